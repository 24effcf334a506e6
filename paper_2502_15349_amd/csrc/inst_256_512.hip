// Retention in its parallel form at D_qk = 256, D_v = 512 (Table 2, "Retention Parallel"): a kernel of its own, because the
// output accumulators of 512 columns do not fit a wavefront's registers beside the queries.
//
// As four passes of the 256 / 128 kernel, one per 128 value columns, every score was formed four times (twice the matrix
// instructions of the operation itself), and every wavefront read all keys of a tile for its own 32 rows: the reads took the LDS as
// long as the products took the matrix units.  Here a workgroup owns 128 query rows and all 512 columns:
//   * 8 wavefronts: two row groups of 64 rows, four wavefronts each, one per 128 value columns: 64 x 128 accumulators are 128
//     registers, and a value fragment read from LDS serves two products;
//   * the scores of a row group's 64 rows against a tile of 32 keys are formed once, in four parts of 16 keys x 32 rows (16 x 16 x 32
//     products: 32 rows of Q are 64 registers), one per wavefront; the weights go to the others through LDS in bf16, as they enter
//     the second product anyway, in its register order.
// Per 32 keys a wavefront issues 16 small and 16 large products (768 clocks, 1536 for the two on a SIMD) and reads 20 KB of LDS
// (640 clocks for all eight at 256 bytes per clock).  The scores of the next tile come first in a step, its weights are formed between the
// products of this tile's values, and a step ends with the one barrier, which hands over the weights, the tiles that have landed and
// the stages that are free.
// Measured, four passes / this kernel (us): 1 x 32 heads x 4096 691 / 420 (bf16 output 675 / 404), 1 x 32/8 x 2048 258 / 113, 2 x 24/6 x 3001 765 /
// 435, 1 x 16 x 300 68 / 21.  A step takes 2900 to 3000 clocks, about twice its products.  What did not move that: key fragments four, six
// or eight ahead, the first value fragments requested early, the row groups in opposite order (weights not between products:
// 428); fewer instructions did a little (running copy addresses: 425 -> 422), and a kernel that spills a single fragment
// loses a tenth (its reload waits for the copies).
#include "dispatch.hpp"

#include "attn_bwd_kernel.hpp"  // read_tr_frag

namespace ae {
namespace {

template <int NORM_>
struct WideCfg {
  static constexpr int DQK = 256, DV = 512, NORM = NORM_, MOD = MOD_DECAY, MASK = 1;
  static constexpr bool FOLD = false;
  static constexpr int THREADS = 512, BLOCK_M = 128, BLOCK_N = 32;
  static constexpr int RB_K = DQK * 2, RB_V = DV * 2, K_BYTES = BLOCK_N * RB_K, V_BYTES = BLOCK_N * RB_V, STAGES = 3;
  static constexpr int P_BYTES = BLOCK_M * BLOCK_N * 2;  // the weights of a tile, two buffers
  static constexpr int kV = STAGES * K_BYTES, kP = kV + STAGES * V_BYTES, LDS_BYTES = kP + 2 * P_BYTES;
  static constexpr int kSums = 8 * 32 * 128 * 4;         // at the end: output blocks, then the row sums
  static_assert(LDS_BYTES <= 160 * 1024 && kSums + 1024 <= LDS_BYTES, "tiles do not fit LDS");
};

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

template <class C>
__global__ __launch_bounds__(C::THREADS, 2) void attn_fwd_wide_kernel(const Params p, const DecayTable dt) {
  __shared__ __attribute__((aligned(1024))) char smem[C::LDS_BYTES];
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_char*)smem);
  // workgroup -> (batch, kv head, q head, q tile): as in attn_fwd_kernel
  int group, t_in;
  if (!place_in_group(blockIdx.x, p.n_groups, p.n_qtiles * p.g, p.interleave, p.cut, group, t_in)) return;
  const int b = group / p.H_kv, hkv = group % p.H_kv;
  const int hq = hkv * p.g + (t_in % p.g), qtile = p.n_qtiles - 1 - t_in / p.g;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rg = wave >> 2, cw = wave & 3;  // row group; 128 value columns
  const int kh = cw & 1, qh = cw >> 1;      // part of the scores: 16 of the 32 keys, 32 of the 64 rows
  const int l16 = lane & 15, g4 = lane >> 4, l32 = lane & 31, half = lane >> 5;
  const int off = p.L_k - p.L_q, i_wg = qtile * C::BLOCK_M, i_rg = i_wg + 64 * rg;
  const __bf16* kbase = p.K + b * p.ks[0] + hkv * p.ks[1];
  const __bf16* vbase = p.V + b * p.vs[0] + hkv * p.vs[1];
  const float g2 = dt.log2_gamma[hq], c = p.neg_q ? -p.c : p.c;

  // keys the workgroup walks, and those of them that some row of this row group sees
  const int kmax = max(0, min(p.L_k, i_wg + C::BLOCK_M + off)), kmax_rg = i_rg < p.L_q ? max(0, min(p.L_k, i_rg + 64 + off)) : 0;
  const int n_tiles = (kmax + C::BLOCK_N - 1) / C::BLOCK_N, n_rg = (kmax_rg + C::BLOCK_N - 1) / C::BLOCK_N;
  // ... and that some row of its first 32 sees: as many tiles or one less.  Weight 0 times an infinite value is NaN, so rows meet no
  // value rows behind the tile that their block of 32 ends in, as in attn_fwd_kernel.
  const int kmax_32 = i_rg < p.L_q ? max(0, min(p.L_k, i_rg + 32 + off)) : 0, n_32 = (kmax_32 + C::BLOCK_N - 1) / C::BLOCK_N;

  // ---- copies: a wavefront moves blocks wave and wave + 8 of a K tile (two rows each) and rows wave + 8 i of a V tile ----
  // (16-byte chunk k of row r stands at k ^ (r % 16) in a K tile, at k ^ 4 (r % 4) in a V tile)
  int ln = lane;  // (the loop's own copy, see there)
  // (kp, vp: the first row of the tile that goes next, kt, vt its number; past the last tile the last one again, to a stage
  // that nobody reads)
  const char* kp = reinterpret_cast<const char*>(kbase);
  const char* vp = reinterpret_cast<const char*>(vbase);
  const int64_t ktile = (int64_t)C::BLOCK_N * p.ks[2] * 2, vtile = (int64_t)C::BLOCK_N * p.vs[2] * 2;
  const uint32_t krb = (uint32_t)p.ks[2] * 2u, vrb = (uint32_t)p.vs[2] * 2u;
  int kt = 0, vt = 0;
  auto copy_k = [&](auto ic, uint32_t stage) {
    constexpr int i = decltype(ic)::value;
    const int krow = 2 * wave + (ln >> 5), r = min(krow + 16 * i, p.L_k - 1 - kt * C::BLOCK_N);
    dma16_at<i * 8192>(kp, (uint32_t)r * krb + (uint32_t)((ln & 31) ^ krow) * 16u, lds0 + stage * C::K_BYTES + wave * 1024);
    if constexpr (i == 1)
      if (kt + 1 < n_tiles) {
        kp += ktile;
        ++kt;
      }
  };
  auto copy_v = [&](auto ic, uint32_t stage) {
    constexpr int i = decltype(ic)::value;
    const uint32_t r = (uint32_t)min(wave + 8 * i, p.L_k - 1 - vt * C::BLOCK_N);
    dma16_at<i * 8192>(vp, r * vrb + (uint32_t)((ln ^ (4 * (wave & 3))) * 16), lds0 + C::kV + stage * C::V_BYTES + wave * 1024);
    if constexpr (i == 3)
      if (vt + 1 < n_tiles) {
        vp += vtile;
        ++vt;
      }
  };
  auto whole_k = [&](uint32_t stage) { static_for<0, 2>([&](auto ic) { copy_k(ic, stage); }); };
  auto whole_v = [&](uint32_t stage) { static_for<0, 4>([&](auto ic) { copy_v(ic, stage); }); };
  constexpr int kCopies = 6;  // instructions per tile

  // ---- queries: two blocks of 16 rows, B fragments ----
  bf16x8 qf[2][8];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const int row = min(i_rg + 32 * qh + 16 * n + l16, p.L_q - 1);
    const __bf16* src = p.Q + b * p.qs[0] + hq * p.qs[1] + (int64_t)row * p.qs[2] + 8 * g4;
#pragma unroll
    for (int t = 0; t < 8; ++t) qf[n][t] = *reinterpret_cast<const bf16x8*>(src + 32 * t);
  }
  if (n_tiles > 0) {
    whole_k(0);
    whole_v(0);
    whole_k(1);
    whole_v(1);
    whole_k(2);
  }
  // (consumed here once: inside the loop the compiler would wait for these loads, and so for the copies, see attn_bwd_kernel.hpp)
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int t = 0; t < 8; ++t) pin(qf[n][t]);

  f32x16 o[2][4];  // O^T: 32 rows (columns of the tile) x 32 value columns each
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) o[q][v] = zero16();
  float sum[2] = {0.f, 0.f};

  // ---- fragment addresses inside stage 0 (the registers are full: of each kind one, the others differ by a bit pattern) ----
  uint32_t ka = lds0 + (16 * kh + l16) * C::RB_K + ((g4 ^ l16) << 4);  // 32 columns further on: ^ 64 n, n < 4, then + 256
  // row 4 half + l16 / 4 of the transposing read, four columns lane % 4 of 16; 32 columns further on: ^ 64 n
  uint32_t va = lds0 + C::kV + (4 * half + (l16 >> 2)) * C::RB_V + (((16 * cw + 2 * (g4 & 1) + ((lane & 3) >> 1)) ^ (4 * (l16 >> 2))) << 4) + 8 * (lane & 1);
  // weights: row of 64 bytes per query, chunk 2 s + h = keys 16 s + 8 a + 4 h + {0..3}, a = 0, 1, at chunk ^ (row / 4 % 4);
  // the second 16-key step: ^ 32; the second block of 16 queries: + 1024
  const uint32_t pbase = lds0 + C::kP + rg * (C::P_BYTES / 2);
  uint32_t pr = pbase + l32 * 64 + ((half ^ ((l32 >> 2) & 3)) << 4);
  uint32_t pw = pbase + (32 * qh + l16) * 64 + (((2 * kh + (g4 & 1)) ^ ((l16 >> 2) & 3)) << 4) + 8 * (g4 >> 1);

  f32x4 sc[2];
  bf16x8 vr4[4], pf[2];  // the next V and weight fragments
  auto v_frag = [&](int n, uint32_t so) {  // 16-key step n / 4, value columns 32 (n % 4) ..
    const uint32_t a = ((va + so) ^ (64u * (n % 4))) + (n / 4) * 16 * C::RB_V;
    return read_tr_frag(a, a + 8 * C::RB_V);
  };
  // Scores of the tile in K stage su; behind its last key fragments the first ones that values() needs are requested.
  // (the copies go out one instruction at a time between the products: queued together they hold up every wavefront at the
  // compute unit's memory pipe; k_copy, v_copy: issues instruction number ic of the step's)
  auto scores = [&](auto aheadc, uint32_t su, uint32_t sv, auto&& k_copy) {
    constexpr bool AHEAD = decltype(aheadc)::value;
    constexpr int RING = 8;
    const uint32_t so = su * C::K_BYTES;
    auto k_frag = [&](int n) { return read_k_frag(((ka + so) ^ (64u * (n % 4))) + (n / 4) * 256); };
    bf16x8 ring[RING];
#pragma unroll
    for (int n = 0; n < RING; ++n) ring[n] = k_frag(n);
    sched_fence();
    sc[0] = sc[1] = (f32x4){0.f, 0.f, 0.f, 0.f};
    static_for<0, 8>([&](auto nc) {
      constexpr int n = decltype(nc)::value;
      sc[0] = mfma16(ring[n % RING], qf[0][n], sc[0]);
      sc[1] = mfma16(ring[n % RING], qf[1][n], sc[1]);
      if constexpr (n + RING < 8) ring[n % RING] = k_frag(n + RING);
      if constexpr (AHEAD && n >= 6) vr4[n - 6] = v_frag(n - 6, sv * C::V_BYTES);
      sched_fence();
      if constexpr (n % 4 == 1) k_copy(std::integral_constant<int, n / 4>{});
    });
  };
  // weights of tile u from its scores, to buffer u % 2: register r is key 32 u + 16 kh + 4 g4 + r, the lane's query l16 of block n
  auto weights = [&](auto nc, int u) {
    constexpr int n = decltype(nc)::value;
    const int i0 = i_rg + 32 * qh + off, d0 = i0 + 16 * n + (ln & 15) - u * C::BLOCK_N - 16 * kh - 4 * (ln >> 4);
    const bool masked = (u + 1) * C::BLOCK_N > p.L_k || (u + 1) * C::BLOCK_N - 1 > i0;
    float x[4];
    const float base = g2 * (float)d0;
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = sc[n][r] * c * fast_exp2(__builtin_fmaf(-g2, (float)r, base));
    if (masked) {
      const int lim = min(d0, p.L_k - 1 - u * C::BLOCK_N - 16 * kh - 4 * (ln >> 4));
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = r > lim ? 0.f : x[r];
    }
    if constexpr (C::NORM == NORM_ABSSUM) sum[n] += (fabsf(x[0]) + fabsf(x[1])) + (fabsf(x[2]) + fabsf(x[3]));
    if constexpr (C::NORM == NORM_ABS_OF_SUM) sum[n] += (x[0] + x[1]) + (x[2] + x[3]);
    bf16x4 h;
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = (__bf16)x[r];
    *reinterpret_cast<__attribute__((address_space(3))) bf16x4*>((lds_char*)(uintptr_t)(pw + n * 1024 + (u & 1) * C::P_BYTES)) = h;
  };
  // O^T += V^T P^T for tile t; between the products, the weights of tile t + 1 (behind the last tile: none are visible, all are 0)
  auto values = [&](int t, uint32_t sv, auto&& v_copy) {
#pragma unroll
    for (int q = 0; q < 2; ++q) pf[q] = read_k_frag(pr + (t & 1) * C::P_BYTES + q * 2048);
    vr4[2] = v_frag(2, sv * C::V_BYTES);
    vr4[3] = v_frag(3, sv * C::V_BYTES);
    sched_fence();
    static_for<0, 8>([&](auto nc) {
      constexpr int n = decltype(nc)::value;
      o[0][n % 4] = mfma(vr4[n % 4], pf[0], o[0][n % 4]);
      o[1][n % 4] = mfma(vr4[n % 4], pf[1], o[1][n % 4]);
      if constexpr (n + 4 < 8) vr4[n % 4] = v_frag(n + 4, sv * C::V_BYTES);
      if constexpr (n == 3) {
#pragma unroll
        for (int q = 0; q < 2; ++q) pf[q] = read_k_frag((pr ^ 32u) + (t & 1) * C::P_BYTES + q * 2048);
      }
      sched_fence();
      if constexpr (n % 2 == 0) v_copy(std::integral_constant<int, n / 2>{});
      if constexpr (n == 1 || n == 4) weights(std::integral_constant<int, n / 4>{}, t + 1);
      sched_fence();
    });
  };
  // the same for the second 32 rows of the row group alone, for its last tile (behind which no weights are wanted)
  auto values_of_second = [&](int t, uint32_t sv) {
    static_for<0, 8>([&](auto nc) {
      constexpr int n = decltype(nc)::value;
      if constexpr (n % 4 == 0) pf[1] = read_k_frag((pr ^ (8u * n)) + (t & 1) * C::P_BYTES + 2048);
      o[1][n % 4] = mfma(v_frag(n, sv * C::V_BYTES), pf[1], o[1][n % 4]);
      sched_fence();
    });
  };
  auto next = [](uint32_t s) { return s == C::STAGES - 1 ? 0u : s + 1; };

  if (n_tiles > 0) {
    // tile 0 of K has landed (the copies behind it: V 0, K 1, V 1, K 2)
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * kCopies) : "memory");
    if (n_rg > 0) {
      scores(std::false_type{}, 0, 0, [](auto) {});
      weights(std::integral_constant<int, 0>{}, 0);
      weights(std::integral_constant<int, 1>{}, 0);
    }
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kCopies) : "memory");
    // Step t of the walk: V of tile t, K of tile t + 1 and the weights of tile t are there for all, and every wavefront is done with
    // K of tile t and V of tile t - 1, whose stages take K of tile t + 3 and V of tile t + 2.
    uint32_t st = 0;  // t % 3
    auto step = [&](auto&& work) {
      const uint32_t st1 = next(st), st2 = next(st1);
      // (hidden from the optimiser: what is derived from these is formed where it is used, not kept through the loop: registers)
      pin(ka);
      pin(va);
      pin(pr);
      pin(pw);
      pin(ln);
      work(st1, st2);
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kCopies) : "memory");
      st = st1;
    };
    int t = 0;
#pragma clang loop unroll(disable)
    for (; t < n_32; ++t)
      step([&](uint32_t st1, uint32_t st2) {
        scores(std::true_type{}, st1, st, [&](auto ic) { copy_k(ic, st); });
        values(t, st, [&](auto ic) { copy_v(ic, st2); });
      });
#pragma clang loop unroll(disable)
    for (; t < n_tiles; ++t)
      step([&](uint32_t, uint32_t st2) {
        whole_k(st);
        whole_v(st2);
        if (t < n_rg) values_of_second(t, st);
      });
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");  // the LDS of the tiles is free
  }

  // ---- row sums: over the four quarters of a 16-key part, then the two parts ----
  float inv[2] = {1.f, 1.f};
  if constexpr (C::NORM != NORM_NONE) {
    const uint32_t sums = lds0 + C::kSums + rg * 512;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      sum[n] += __shfl_xor(sum[n], 16);
      sum[n] += __shfl_xor(sum[n], 32);
      if (g4 == 0) lds_store4(sums + (64 * kh + 32 * qh + 16 * n + l16) * 4, sum[n]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float l = lds_read4(sums + (32 * q + l32) * 4) + lds_read4(sums + (64 + 32 * q + l32) * 4);
      inv[q] = 1.f / fmaxf(C::NORM == NORM_ABS_OF_SUM ? fabsf(l) : l, 1.f);
      const int i = i_rg + 32 * q + l32;
      if (p.stats != nullptr && cw == 0 && half == 0 && i < p.L_q) p.stats[((int64_t)b * p.H_q + hq) * p.L_q + i] = l;
    }
  }
  // ---- store: 32 rows x 128 columns at a time, turned around in the wavefront's own 16 KB of LDS (chunk k of row r at k ^ (r % 16)) ----
  const int64_t head = b * p.os[0] + hq * p.os[1];
  const uint32_t obuf = lds0 + wave * 16384;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = o[q][v][4 * r4 + e] * inv[q];
        lds_write16(obuf + l32 * 512 + (((8 * v + 2 * r4 + half) ^ (l32 & 15)) << 4), x);
      }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int row = 2 * k + half, i = i_rg + 32 * q + row;
      const f32x4 x = lds_read16(obuf + row * 512 + ((l32 ^ (row & 15)) << 4));
      if (i < p.L_q) {
        const int64_t e = head + (int64_t)i * p.os[2] + 128 * cw + 4 * l32;
        if (p.out_bf16) {
          bf16x4 h;
#pragma unroll
          for (int k4 = 0; k4 < 4; ++k4) h[k4] = (__bf16)x[k4];
          *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.O) + e) = h;
        } else {
          *reinterpret_cast<f32x4*>(static_cast<float*>(p.O) + e) = x;
        }
      }
    }
  }
}

template <class C>
hipError_t launch_wide(const Params& p, const DecayTable& dt, int grid, hipStream_t s) {
  hipLaunchKernelGGL(attn_fwd_wide_kernel<C>, dim3(grid), dim3(C::THREADS), 0, s, p, dt);
  return hipGetLastError();
}
template <int NORM>
constexpr KernelEntry wide_entry(const char* name) {
  typedef WideCfg<NORM> C;
  return KernelEntry{C::DQK, C::DV, C::NORM, C::MOD, C::MASK, 0, C::BLOCK_M, C::BLOCK_N, C::THREADS, C::LDS_BYTES, &launch_wide<C>, name};
}

}  // namespace

// (the names: 128 value columns per wavefront, four wavefronts)
static const KernelEntry kTable[] = {wide_entry<NORM_ABSSUM>("attn_fwd_wide<256,128x4,NORM_ABSSUM,MOD_DECAY,true>"),
                                     wide_entry<NORM_ABS_OF_SUM>("attn_fwd_wide<256,128x4,NORM_ABS_OF_SUM,MOD_DECAY,true>"),
                                     wide_entry<NORM_NONE>("attn_fwd_wide<256,128x4,NORM_NONE,MOD_DECAY,true>")};

const KernelEntry* table_256_512(int* n) {
  *n = (int)(sizeof(kTable) / sizeof(kTable[0]));
  return kTable;
}
}  // namespace ae
