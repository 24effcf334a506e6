// Decoding shapes (paper Table 2, the decoding row: one query row per head against thousands of keys; Section 4.1,
// online row-norm interface: the state of two key blocks is combined by the rule of the online softmax).  One query row
// has no use for a 256-row tile: the work is reading K and V once, so the kernel is a stream.  A workgroup owns one
// (batch, k/v head, key range) and up to G of the q heads that share it, and its W wavefronts take the range's keys
// four at a time; 16 lanes share a key, each holding D / 16 consecutive elements of its row (one 16-byte load per lane
// for 128 elements, an 8-byte one more for 192), so every load instruction of a wavefront reads four whole rows,
// contiguous in memory.  The dot product is D / 16 multiply-adds and four data-parallel-primitive adds inside the row of
// 16 lanes; every group of 16 lanes keeps an online softmax state of its own per q head (reference, sum, D_v / 16 output
// columns), and the 4 W states of a workgroup are combined at the end into one normalised row: the result, where the keys
// are one range (DIRECT), or else a partial row and its log-sum-exp, which attn_merge_kernel combines over the key
// ranges.  Loads run one block of kDecodeDepth steps ahead of the arithmetic (registers only, no LDS tiles, no barrier
// inside the loop).
//
// What bounds it: HBM with one q head per k/v head (32 x 16 heads x 4096 keys, 192/128: 6.1 TB/s); with more, the vector
// arithmetic per key and head, about 30 instructions for 16 lanes (64 x 32/8 heads x 1000 keys, 128/128: 4.8 TB/s).
// Scoring the heads of a block of keys first and rescaling once per block saves a quarter of them and costs the registers
// of a second workgroup per compute unit (16 x 32/8 x 5003: 88 -> 99 us).  Keys in one range were the 256-row
// attention kernel's before, one workgroup per q head: 16 x 32/8 heads x 5003 keys 144 -> 75 us, 64 x 32/8 x 1000
// 154 -> 54 us, 1 x 16 x 8192 (192/128) 127 -> 73 us, 1 x 12 x 300 (64/64) 8.1 -> 5.0 us.
#include <hip/hip_runtime.h>

#include "attn_decode.hpp"

namespace ae {
namespace {

constexpr int kDecodeDepth = 4;  // steps (of 4 keys per wavefront) loaded ahead

template <int N>
struct RowPiece {  // N bf16 elements of a row, N = 4, 8 or 12
  uint32_t w[N / 2];
};

template <int N>
__device__ __forceinline__ RowPiece<N> load_piece(const __bf16* row, int sub) {
  RowPiece<N> r;
  if constexpr (N == 4) {
    const uint2 a = *reinterpret_cast<const uint2*>(row + 4 * sub);
    r.w[0] = a.x, r.w[1] = a.y;
  } else {
    const uint4 a = *reinterpret_cast<const uint4*>(row + 8 * sub);
    r.w[0] = a.x, r.w[1] = a.y, r.w[2] = a.z, r.w[3] = a.w;
    if constexpr (N == 12) {
      const uint2 b = *reinterpret_cast<const uint2*>(row + 128 + 4 * sub);
      r.w[4] = b.x, r.w[5] = b.y;
    }
  }
  return r;
}

// element e of a piece as fp32 (bf16 is the upper half of an fp32)
template <int N>
__device__ __forceinline__ float elem(const RowPiece<N>& r, int e) {
  const uint32_t w = r.w[e / 2];
  return __builtin_bit_cast(float, (e & 1) ? (w & 0xffff0000u) : (w << 16));
}

// sum over the 16 lanes of a row, left in every one of them
__device__ __forceinline__ float row16_sum(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xb1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4e, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xf, 0xf, false));  // row_half_mirror
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x140, 0xf, 0xf, false));  // row_mirror
  return x;
}

constexpr float kNone = -1e30f;  // "no key yet": finite, so that differences of references stay finite

// G: q heads of the k/v head that one workgroup serves, all from one pass over the keys.
template <int DQK, int DV, int G, bool DIRECT, int W>
__global__ __launch_bounds__(64 * W) void attn_decode_kernel(const DecodeParams p) {
  constexpr int NK = DQK / 16, NV = DV / 16;
  // one q head: the states of all rows of 16 lanes meet in LDS; more: one per wavefront, folded in registers before
  constexpr int NS = G == 1 ? 4 * W : W;
  __shared__ float red[NS][G][DV + 2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = lane >> 4, sub = lane & 15;
  // (key range, batch, k/v head) fastest: the workgroups of one k/v head that serve different q heads are a multiple
  // of 8 apart where that number is one, and then run on the same XCD
  // Sets of G q heads slowest: the workgroups that read the same keys for different sets are `units` apart, and run on
  // the same XCD where that is a multiple of 8 (they take the keys from its L2 then; one q head per workgroup, 32 q
  // on 8 k/v heads x 4096 keys in 6 ranges: 19.1 us with the sets fastest, 16.5 so).
  const int set = blockIdx.x / p.units, unit = blockIdx.x % p.units, head = unit / p.n_splits;
  const int c = unit % p.n_splits;
  const int b = head / p.H_kv, hk = head % p.H_kv;  // batch entry, k/v head
  const int h0 = hk * p.g + set * G, n_heads = G == 1 ? 1 : min(G, p.g - set * G);
  const int j_begin = c * p.split_keys, j_end = min(p.L_k, j_begin + p.split_keys);
  const __bf16* Kh = p.K + b * p.ks[0] + hk * p.ks[1];
  const __bf16* Vh = p.V + b * p.vs[0] + hk * p.vs[1];

  // the query rows, in log2 units: scale * log2(e) * q, fp32 (a head past the group repeats the last one)
  float q[G][NK];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const RowPiece<NK> qp = load_piece<NK>(p.Q + b * p.qs[0] + (h0 + min(h, n_heads - 1)) * p.qs[1], sub);
#pragma unroll
    for (int e = 0; e < NK; ++e) q[h][e] = elem(qp, e) * p.c;
  }
  float m[G], l[G], acc[G][NV];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    m[h] = kNone;
    l[h] = 0.f;
#pragma unroll
    for (int e = 0; e < NV; ++e) acc[h][e] = 0.f;
  }

  // step s of this wavefront: keys j_begin + (W s + wave) * 4 + grp
  const int n_steps = (j_end - j_begin + 4 * W - 1) / (4 * W);
  auto key_of = [&](int s) { return j_begin + (W * s + wave) * 4 + grp; };
  RowPiece<NK> kbuf[2][kDecodeDepth];
  RowPiece<NV> vbuf[2][kDecodeDepth];
  auto issue = [&](int s0, int which) {
#pragma unroll
    for (int u = 0; u < kDecodeDepth; ++u) {
      const int j = min(key_of(s0 + u), p.L_k - 1);  // (keys past the end are read as the last key and get weight 0)
      kbuf[which][u] = load_piece<NK>(Kh + (int64_t)j * p.ks[2], sub);
      vbuf[which][u] = load_piece<NV>(Vh + (int64_t)j * p.vs[2], sub);
    }
  };
  auto work = [&](int s0, int which) {
#pragma unroll
    for (int u = 0; u < kDecodeDepth; ++u) {
      const bool live = key_of(s0 + u) < j_end;
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float x = 0.f;
#pragma unroll
        for (int e = 0; e < NK; ++e) x = __builtin_fmaf(q[h][e], elem(kbuf[which][u], e), x);
        x = row16_sum(x);
        asm volatile("" : "+v"(x));  // (or the compiler makes a branch of the selection, with the multiply-adds inside)
        x = live ? x : kNone;
        const float mn = fmaxf(m[h], x);
        const float alpha = __builtin_amdgcn_exp2f(m[h] - mn);          // 1 while the reference stands
        const float w = live ? __builtin_amdgcn_exp2f(x - mn) : 0.f;
        m[h] = mn;
        l[h] = l[h] * alpha + w;
#pragma unroll
        for (int e = 0; e < NV; ++e) acc[h][e] = __builtin_fmaf(w, elem(vbuf[which][u], e), acc[h][e] * alpha);
      }
    }
  };
  // blocks of kDecodeDepth steps, the loads of block n + 1 in flight while block n is worked on
  const int n_blocks = (n_steps + kDecodeDepth - 1) / kDecodeDepth;
  if (n_blocks > 0) issue(0, 0);
  for (int n = 0; n < n_blocks; n += 2) {
    if (n + 1 < n_blocks) issue((n + 1) * kDecodeDepth, 1);
    work(n * kDecodeDepth, 0);
    if (n + 1 < n_blocks) {
      if (n + 2 < n_blocks) issue((n + 2) * kDecodeDepth, 0);
      work((n + 1) * kDecodeDepth, 1);
    }
  }

  // ---- the states of the workgroup (W wavefronts x 4 rows of lanes) into one per q head ----
#pragma unroll
  for (int h = 0; h < G; ++h) {
    if constexpr (G > 1) {
      auto fold = [&](int ofs) {
        const float mo = __shfl_xor(m[h], ofs), mn = fmaxf(m[h], mo);
        const float fa = __builtin_amdgcn_exp2f(m[h] - mn), fb = __builtin_amdgcn_exp2f(mo - mn);
        l[h] = l[h] * fa + __shfl_xor(l[h], ofs) * fb;
#pragma unroll
        for (int e = 0; e < NV; ++e) acc[h][e] = acc[h][e] * fa + __shfl_xor(acc[h][e], ofs) * fb;
        m[h] = mn;
      };
      fold(16);
      fold(32);
    }
    if (G == 1 || grp == 0) {
      float* mine = red[G == 1 ? 4 * wave + grp : wave][h];
#pragma unroll
      for (int e = 0; e < NV; ++e) mine[NV * sub + e] = acc[h][e];
      if (sub == 0) {
        mine[DV] = m[h];
        mine[DV + 1] = l[h];
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n_heads * DV; i += 64 * W) {
    const int h = i / DV, d = i % DV;
    float M = kNone;
#pragma unroll
    for (int s = 0; s < NS; ++s) M = fmaxf(M, red[s][h][DV]);
    float L = 0.f, o = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const float f = __builtin_amdgcn_exp2f(red[s][h][DV] - M);
      L += f * red[s][h][DV + 1];
      o += f * red[s][h][d];
    }
    // no visible key leaves the sum at +0; a NaN sum (a NaN or infinite score) makes the row NaN.  The two are told apart by
    // their bits: device code is compiled under the assumption that no NaN occurs, which a comparison of floats may use
    const bool any = __builtin_bit_cast(uint32_t, L) != 0;
    o = any ? o / L : 0.f;
    // (a constant bias is in every weight of the row and leaves the output alone: only the statistic sees it, here where the
    // keys are one range, in the merge kernel where they are several.  Added to the scores instead, a bias of 1e6 costs their
    // fraction and one beyond -7e29 the whole row)
    const float lse = any ? (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f + (DIRECT ? p.bias : 0.f) : -INFINITY;
    const int64_t row = (int64_t)b * p.H_q + h0 + h;
    if constexpr (!DIRECT) {
      p.ws_o[((int64_t)c * p.rows + row) * DV + d] = o;
      if (d == 0) p.ws_lse[(int64_t)c * p.rows + row] = lse;
    } else {
      const int64_t at = b * p.os[0] + (h0 + h) * p.os[1] + d;
      if (p.out_bf16) static_cast<__bf16*>(p.O)[at] = (__bf16)o;
      else static_cast<float*>(p.O)[at] = o;
      if (d == 0 && p.stats != nullptr) p.stats[row] = lse;
    }
  }
}

template <int DQK, int DV, int G, int W>
hipError_t launch_waves(const DecodeParams& p, unsigned grid, hipStream_t s) {
  if (p.n_splits > 1) hipLaunchKernelGGL((attn_decode_kernel<DQK, DV, G, false, W>), dim3(grid), dim3(64 * W), 0, s, p);
  else hipLaunchKernelGGL((attn_decode_kernel<DQK, DV, G, true, W>), dim3(grid), dim3(64 * W), 0, s, p);
  return hipGetLastError();
}

constexpr int64_t kUnits = 256;  // compute units

template <int DQK, int DV, int G>
hipError_t launch_heads(const DecodeParams& p, hipStream_t s) {
  const int64_t grid = p.rows / p.g * ((p.g + G - 1) / G) * p.n_splits;
  if (!launch_fits(grid, 256)) return hipErrorInvalidValue;  // (more wavefronts only for few workgroups, see below)
  DecodeParams q = p;
  q.units = (int)(p.rows / p.g * p.n_splits);
  // Eight wavefronts instead of four keep more loads in flight and halve a workgroup's walk; taken where no compute unit has a
  // second workgroup to do that, from 320 keys on.  128/128, us, 4 / 8 wavefronts: 4 x 16 heads x 4096 keys (64 workgroups) 46 / 37,
  // 16 x 32/8 x 4096 (256 of two heads) 64 / 55, 16 x 64/8 x 4096 (256 of four) 98 / 89; against it 17 x 16 x 4096 (272 workgroups,
  // 64/64) 61 / 67, 33 x 64/8 x 300 (264 of eight) 32 / 42.  Not for 192-element keys that no other workgroup of the XCD reads,
  // once 128 workgroups pull them from HBM: 12 x 16 x 1000 25.8 / 26.9, 2 x 16 x 8192 in 8 ranges 30.4 / 32.9, 12 x 16 x 8192
  // 172 / 186, 17 x 8/1 x 16384 200 / 222 (shared ones: 4 x 32/8 x 8192 in 2 ranges 55 / 45).
  const bool from_hbm = DQK == 192 && G == 1 && (p.g == 1 || q.units % 8 != 0) && grid >= 128;
  const bool wide = grid <= kUnits && p.split_keys >= 320 && !from_hbm;
  return wide ? launch_waves<DQK, DV, G, 8>(q, (unsigned)grid, s) : launch_waves<DQK, DV, G, 4>(q, (unsigned)grid, s);
}

// How many of the q heads of a k/v head one workgroup serves.  A key costs a workgroup its loads and, per head, its arithmetic,
// about as 5 to 2, a head its place in the combination at the end, about what the loads of 128 keys cost, and the fullest compute
// unit decides: the G that makes rounds of 256 workgroups x (keys (5 + 2 G) + 640 G) least.  Over batch 1 to 64, 300 to 32k keys, 1
// to 32 ranges, 1, 3, 4 and 8 q heads per k/v head and the three head dims (2112 shapes) the times are 0.7 % above the best G and
// number of wavefronts on the average; with the most heads that leave 256 workgroups it was 4.1 %.
// 128/128, 32/8 heads x 4096 keys, us with 1 / 2 / 4 heads: batch 12 65 / 52 / 87, 15 73 / 54 / 88, 16 77 / 55 / 89, 17 114 / 100 / 91.
// D_qk = 192 with eight needs 318 registers and stops at four.
template <int DQK, int DV>
hipError_t launch(const DecodeParams& p, hipStream_t s) {
  const int64_t units = p.rows / p.g * p.n_splits;
  int best = 1;
  int64_t least = INT64_MAX;
  for (int G = 1; G <= (DQK <= 128 ? 8 : 4) && G < 2 * p.g; G *= 2) {
    const int64_t rounds = (units * ((p.g + G - 1) / G) + kUnits - 1) / kUnits;
    const int64_t cost = rounds * ((int64_t)p.split_keys * (5 + 2 * G) + 640 * G);
    if (cost < least) {
      least = cost;
      best = G;
    }
  }
  if constexpr (DQK <= 128)
    if (best == 8) return launch_heads<DQK, DV, 8>(p, s);
  if (best == 4) return launch_heads<DQK, DV, 4>(p, s);
  if (best == 2) return launch_heads<DQK, DV, 2>(p, s);
  return launch_heads<DQK, DV, 1>(p, s);
}

}  // namespace

bool decode_supported(int dqk, int dv) { return (dqk == 64 && dv == 64) || (dqk == 128 && dv == 128) || (dqk == 192 && dv == 128); }

hipError_t launch_decode(const DecodeParams& p, int dqk, int dv, hipStream_t s) {
  if (p.n_splits < 1 || p.split_keys < 1 || p.rows < 1) return hipErrorInvalidValue;
  if (dqk == 64 && dv == 64) return launch<64, 64>(p, s);
  if (dqk == 128 && dv == 128) return launch<128, 128>(p, s);
  if (dqk == 192 && dv == 128) return launch<192, 128>(p, s);
  return hipErrorInvalidValue;
}

}  // namespace ae
