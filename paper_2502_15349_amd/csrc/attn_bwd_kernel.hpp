// Backward pass of fused parallel-pattern attention for gfx950 (CDNA4): the gradients
// of O = normalization(modification(Q K^T)) V with respect to Q, K and V, for a given
// upstream gradient dO, with the weights recomputed from the row statistic that the
// forward pass keeps (paper Section 4.1, online row-norm interface: the backward graph
// is derived from the same definition and reads the final row scales).
//
//   P   = exp(S' - lse_i)  (softmax)   |  sigmoid(S')            S' = scale * Q K^T + bias
//   dV  = P^T dO                          dP = dO V^T
//   dS' = P * (dP - delta_i), delta_i = dO_i . O_i  (softmax)   |  dP * P * (1 - P)  (sigmoid)
//   no normalization: P = S' or max(S', 0) on visible entries, dS' = dP or dP * [S' > 0]
//   abs-sum family (retention): S' = scale * Q K^T * decay, P = S' / n_i, n_i = max(r_i, 1), r_i = sum_j |S'| or
//     |sum_j S'| (the forward row statistic); dS' = (dP - g * [r_i > 1] * delta_i) / n_i with g = sign(S') or
//     sign(sum_j S'); the gradient of the raw score is dS' * decay
//   dQ  = scale * dS' K                   dK = scale * dS'^T Q
//
// Two sides, in one launch or one each, no atomics, every output written once:
//   * key side (KV_SIDE): a workgroup owns 128 keys of one k/v head and walks the query tiles of
//     the q heads that share it: dK and dV;
//   * query side: a workgroup owns 128 query rows of one q head and walks the key tiles: dQ.
// A wavefront owns 32 rows ("own" side) whose operands it keeps in registers as MFMA B fragments (K, V | Q, dO), and
// the tiles of the other side (Q, dO | K, V) arrive in LDS by global_load_lds.  Per 32 other rows
//   S  [other x own] = Y1 X1^T      dP [other x own] = Y2 X2^T        (bf16 MFMA 32x32x16)
// put a lane's 16 accumulator values in one own column; after the elementwise step they
// are, packed to bf16 and with no data movement, the B operands of
//   dQ^T, dK^T [D_qk x own] += Y1^T dS       dV^T [D_v x own] += Y2^T P
// whose A operands are the same LDS tiles read through the transposing LDS load, in the
// row order that the accumulator layout dictates.
//
// What bounds it is how well a SIMD's vector and matrix work overlap, and that takes two wavefronts per SIMD of at most
// 256 registers.  Where accumulators, resident operands and score tiles of 32 own rows fit that (64/64; 128/128, query
// side), a wavefront does all of the above and two workgroups share a CU: bwd_single_walk.  Where they do not, the 32
// rows go to a pair of wavefronts: bwd_pair_walk (its key side at 128/256 spills up to 4 registers), but for
// short walks, which the first form takes with one workgroup per CU and up to 472 registers.  The lines between the two
// stand in bwd_launch.hpp.
#pragma once
#include "attn_kernel.hpp"

namespace ae {

struct BwdParams {
  const __bf16* Q;
  const __bf16* K;
  const __bf16* V;
  const __bf16* dO;    // [B, H_q, L_q, D_v] contiguous
  const void* O;       // as the forward pass wrote it (softmax only): fp32, or bf16 if o_bf16
  const float* lse;    // [B, H_q, L_q] row statistic of the forward pass (softmax; abs-sum family: r or the signed sum)
  float* delta;        // [B, H_q, L_q] workspace (softmax; abs-sum family: delta where r > 1, signed for |sum|, else 0)
  float* dQ;           // [B, H_q, L_q, D_qk] contiguous fp32
  float* dK;           // [B, H_kv, L_k, D_qk]
  float* dV;           // [B, H_kv, L_k, D_v]
  int B, H_q, H_kv, L_q, L_k, g;
  int o_bf16;
  int64_t qs[3], ks[3], vs[3], os[3];  // element strides {batch, head, row} of Q, K, V, O
  float c2;     // scale * log2(e)
  float b2;     // bias * log2(e)
  float scale;
  // bias-tensor kernels: additive bias per (query, key), bf16, element strides bs[] = {batch, head, row};
  // bunit: log2(e) where the scores are kept in powers of two (softmax, sigmoid), else 1
  const __bf16* bias;
  int64_t bs[3];
  float bunit;
  // optional gradient of the bias tensor, bf16 [B, H_q, L_q, dbias_ld] (per batch and head, not summed over
  // sharers); written by the query-side kernel for the sub-tiles it visits
  __bf16* dbias;
  int64_t dbias_ld;
  // causal kernels: key j is also hidden from query i if j <= i + (L_k - L_q) - window (sliding
  // window); L_q + L_k for the plain causal mask, which hides nothing more
  int window;
  // the handle has a per-head decay: only then is the decay table read (it holds AE_MAX_DECAY_HEADS entries, and
  // handles without decay may have more heads than that)
  int has_decay;
  // (batch, k/v head) groups, or parts of groups, that one XCD walks together, per kernel ([0]: query side, [1]: key side); see the
  // mapping at the top of bwd_single_walk
  int together[2];
  int cut;  // a group's workgroups go to 2^cut XCDs in turn (see group_cut)
};

// Chunk swizzle of the backward tiles.  A tile row is read both ways -- 128-bit row
// fragments, 16 lanes = 16 consecutive rows at a time, and 64-bit transposing loads, 32
// lanes = 4 consecutive rows x 4 chunks at a time -- so the XOR pattern takes 16 values
// over 16 consecutive rows (rows of 128 or 384 bytes alternate between the halves of the
// 256-byte bank window, which supplies one of the four bits) and its upper bits change
// within every aligned group of 4 rows.
template <int CPR>
__device__ __forceinline__ int bswz(int row) {
  return CPR % 16 == 0 ? ((4 * (row & 3)) | ((row >> 2) & 3)) : ((4 * ((row >> 1) & 1)) | ((row >> 2) & 3));
}

// no normalization with the ReLU modification (the forward kernels carry the modification as a
// parameter of its own; here the pair is one more value of the NORM parameter)
constexpr int BWD_NORM_NONE_RELU = 5;
// Abs-sum family, no normalization: the factor between dP and dS' of an entry that is hidden.  A visible entry's is never
// negative, but may be 0 as well where its decay vanishes, and then passes an infinite or NaN dP on, wherever its tile lies.
constexpr float kHiddenFactor = -0.f;
__device__ __forceinline__ bool factor_hidden(float f) { return __builtin_bit_cast(uint32_t, f) == 0x80000000u; }
enum : int { BWD_DQ = 0, BWD_DKV = 1 };  // the query-side kernel (dQ), the key-side kernel (dK and dV)

// ---- one wavefront per 32 own rows ---------------------------------------------------------------------------------
template <int DQK_, int DV_, int NORM_, bool CAUSAL_, int OUT_, bool BIAS_ = false>
struct BwdCfg {
  static constexpr bool BIAS = BIAS_;  // S' = scale * S + bias[b, h_q, i, j]
  static constexpr int DQK = DQK_, DV = DV_, NORM = NORM_, OUT = OUT_;
  static constexpr bool CAUSAL = CAUSAL_, KV_SIDE = OUT_ == BWD_DKV;
  static constexpr int WAVES = 4, THREADS = 256, OWN = 128;  // own rows per workgroup
  static constexpr bool PAIR = false;
  static constexpr int T1 = DQK / 16, T2 = DV / 16;
  static constexpr int DB = DQK / 32;  // 32-row blocks of the transposed result dQ^T / dK^T
  static constexpr bool HAS2 = KV_SIDE;               // key side: a second result, dV^T
  static constexpr int DB2 = HAS2 ? DV / 32 : 0;
  static constexpr int TILE = 64;  // other-side rows per LDS tile (two 32-row sub-tiles)
  static constexpr int RB1 = DQK * 2, RB2 = DV * 2, CPR1 = DQK / 8, CPR2 = DV / 8;
  static constexpr int Y1_BYTES = TILE * RB1, Y2_BYTES = TILE * RB2, STAGE_BYTES = Y1_BYTES + Y2_BYTES;
  // per stage: bias*log2(e) - lse*log2(e) and delta of the tile's rows (key side: they belong to the registers' rows;
  // on the query side they belong to the lane's own row and stay in registers)
  static constexpr int ROW_BYTES = KV_SIDE ? 2 * TILE * 4 : 0;
  // bias tensor: per stage the block of it that the tile meets, 16 KB: [128 own queries][64 keys] on the query
  // side, [64 queries][128 own keys] on the key side
  static constexpr int BIAS_BYTES = BIAS_ ? 16384 : 0;
  static constexpr int LDS_BYTES = 2 * STAGE_BYTES + 2 * ROW_BYTES + 2 * BIAS_BYTES;
  static_assert(NORM == NORM_SOFTMAX || NORM == NORM_SIGMOID || NORM == NORM_NONE || NORM == BWD_NORM_NONE_RELU ||
                    NORM == NORM_ABSSUM || NORM == NORM_ABS_OF_SUM,
                "backward: softmax, sigmoid, the abs-sum family, and no normalization with or without ReLU");
  static constexpr bool ABS = NORM == NORM_ABSSUM || NORM == NORM_ABS_OF_SUM;
  static constexpr bool ROWS = NORM == NORM_SOFTMAX || ABS;  // per-row quantities from the forward statistic and delta
  // no normalization (without ReLU) is the abs-sum form with the row factors fixed at 1 and 0: P = S', dS' = dP,
  // per-head decay included
  static constexpr bool LIN = ABS || NORM == NORM_NONE;
  // Two workgroups per CU (two waves per SIMD, 256 registers each) where the accumulators, the resident operands and the
  // two score tiles leave room for the rest; one (512 registers) otherwise.
  static constexpr bool OCC2 = 16 * (DB + DB2) + 4 * T1 + 4 * T2 + 32 + (BIAS_ ? 8 : 0) <= 176 && LDS_BYTES <= 80 * 1024;
  // one workgroup per CU: the LDS fragments of a step are read as a batch ahead of its MFMAs
  static constexpr bool BATCH = !OCC2 && DQK + DV <= 320;  // (beyond that the batches do not fit 512 registers)
  static_assert(LDS_BYTES <= 160 * 1024, "a workgroup must fit LDS");
  static_assert((TILE * CPR1 / 64) % WAVES == 0 && (TILE * CPR2 / 64) % WAVES == 0, "every wave copies the same number of blocks");
};

__device__ __forceinline__ bf16x8 read_tr_frag(uint32_t addr_lo, uint32_t addr_hi) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)addr_lo);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)addr_hi);
  const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, both);
}

__device__ __forceinline__ bf16x8 pack8(const float (&x)[16], int t) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (__bf16)x[8 * t + e];
  return r;
}

template <class C>
__device__ __forceinline__ void bwd_single_walk(const BwdParams& p, const DecayTable& dt, int block, uint32_t lds0) {
  const uint32_t rows0 = lds0 + 2 * C::STAGE_BYTES;
  const uint32_t bias0 = rows0 + 2 * C::ROW_BYTES;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ln = lane & 31, half = lane >> 5;
  const int off = p.L_k - p.L_q;
  const int L_own = C::KV_SIDE ? p.L_k : p.L_q, L_oth = C::KV_SIDE ? p.L_q : p.L_k;

  // ---- which rows this workgroup owns ----------------------------------------------
  const int n_heads = C::KV_SIDE ? p.H_kv : p.H_q;
  const int n_own_tiles = (L_own + C::OWN - 1) / C::OWN;
  // Workgroups are dealt to the 8 XCDs round-robin, and each XCD has its own L2.  All workgroups of one (batch,
  // k/v head) group -- its own tiles, times the q heads of the group on the query side -- go to one XCD and run
  // there at the same time, `together` groups side by side: they stream the same rows of the other side a few
  // tiles apart, so a tile that one of them pulled into L2 serves the others.  Within a set of groups the
  // workgroups with most work come first (causal).  The grid is padded to whole sets; the surplus exits here.
  int group, item;
  if (!place_in_group(block, p.B * p.H_kv, C::KV_SIDE ? n_own_tiles : n_own_tiles * p.g, p.together[C::KV_SIDE ? 1 : 0], p.cut, group, item)) return;
  const int b = group / p.H_kv, hk = group % p.H_kv;
  int ot = C::KV_SIDE ? item : n_own_tiles - 1 - item / p.g;
  const int ho = C::KV_SIDE ? hk : hk * p.g + item % p.g;  // ho: k/v head (key side) or q head (query side)
  const int own0 = ot * C::OWN, ow0 = own0 + wave * 32;  // first own row of the workgroup / of this wave
  const int own = ow0 + ln;                              // this lane's own row (column of S, dP, G^T)
  const int own_c = own < L_own ? own : L_own - 1;

  // ---- own operands: B fragments, straight from global memory ------------------------
  const __bf16* x1 = C::KV_SIDE ? p.K + b * p.ks[0] + hk * p.ks[1] + (int64_t)own_c * p.ks[2]
                                : p.Q + b * p.qs[0] + ho * p.qs[1] + (int64_t)own_c * p.qs[2];
  const __bf16* x2 = C::KV_SIDE ? p.V + b * p.vs[0] + hk * p.vs[1] + (int64_t)own_c * p.vs[2]
                                : p.dO + (((int64_t)b * p.H_q + ho) * p.L_q + own_c) * C::DV;
  bf16x8 xb1[C::T1], xb2[C::T2];
#pragma unroll
  for (int t = 0; t < C::T1; ++t) xb1[t] = *reinterpret_cast<const bf16x8*>(x1 + (2 * t + half) * 8);
#pragma unroll
  for (int t = 0; t < C::T2; ++t) xb2[t] = *reinterpret_cast<const bf16x8*>(x2 + (2 * t + half) * 8);
  // query side: the row quantities belong to the lane's own row
  // (first: (bias - lse) * log2(e) for softmax, 1 / max(|statistic|, 1) for the abs-sum family; second: delta)
  float nl_own = C::LIN ? 1.f : -INFINITY, dl_own = 0.f;
  if constexpr (!C::KV_SIDE && C::ROWS) {
    if (own < p.L_q) {
      const int64_t r = ((int64_t)b * p.H_q + ho) * p.L_q + own;
      const float st = p.lse[r];
      if constexpr (C::ABS) nl_own = fast_rcp(fmaxf(fabsf(st), 1.f));
      else nl_own = st == -INFINITY ? -INFINITY : p.b2 - st * 1.4426950408889634f;
      dl_own = p.delta[r];
    }
  }
  // Abs-sum family, no normalization: log2 of the decay rate of the q head at hand (0: no decay), and, for sub-tiles whose entries are
  // all visible, what the decay factor of register 4 q + e is of the largest one (register 0 on the key side, 15 on the query side).
  // An exponential and a dozen instructions of index and visibility per entry took the vector unit longer than the products take:
  // 8 x 16 x 4096 causal, 64/64: abs-sum with decay 1457 -> 1185 us, no normalization 1185 -> 871.
  float lg = 0.f, dec_q[C::LIN ? 4 : 1], dec_e[C::LIN ? 4 : 1];
  auto set_decay = [&](int h) {
    if constexpr (C::LIN) {
      lg = p.has_decay ? dt.log2_gamma[h] : 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        dec_q[k] = fast_exp2(lg * (C::KV_SIDE ? 8.f * k : 24.f - 8.f * k));
        dec_e[k] = fast_exp2(lg * (C::KV_SIDE ? 1.f * k : 3.f - k));
      }
    }
  };
  set_decay(C::KV_SIDE ? hk * p.g : ho);

  // ---- the walk over the other side --------------------------------------------------
  // key side: the query tiles from the first one that sees key own0, for each q head of
  // the group; query side: the key tiles up to the last one that row own0 + 127 sees.
  int t_first = 0, t_end = (L_oth + C::TILE - 1) / C::TILE;
  if constexpr (C::CAUSAL) {
    if constexpr (C::KV_SIDE) {
      const int i_first = own0 - off;  // first query that sees key own0
      t_first = i_first > 0 ? i_first / C::TILE : 0;
      if (t_first > t_end) t_first = t_end;
      const int i_last = own0 + C::OWN - 1 - off + p.window - 1;  // last query whose window holds a key here
      const int e = i_last < 0 ? 0 : i_last / C::TILE + 1;
      if (e < t_end) t_end = e;
      if (t_end < t_first) t_end = t_first;
    } else {
      const int j_last = own0 + C::OWN - 1 + off;  // last key any row here may see
      const int e = j_last < 0 ? 0 : j_last / C::TILE + 1;
      if (e < t_end) t_end = e;
      const int j_first = own0 + off - p.window + 1;  // first key inside the window of row own0
      t_first = j_first > 0 ? j_first / C::TILE : 0;
      if (t_first > t_end) t_first = t_end;
    }
  }
  const int nt = t_end - t_first;
  const int total = C::KV_SIDE ? nt * p.g : nt;

  // LDS-DMA maps: block nb of a tile = 64 chunks of 16 bytes, linear in LDS; position ->
  // (row, physical chunk), the logical chunk is the physical one XOR the row's swizzle.
  auto issue_tile = [&](int n, int stage) {
    const int hq = C::KV_SIDE ? hk * p.g + n / nt : ho;
    const int r0 = (t_first + (C::KV_SIDE ? n % nt : n)) * C::TILE;
    const __bf16* y1 = C::KV_SIDE ? p.Q + b * p.qs[0] + hq * p.qs[1] : p.K + b * p.ks[0] + hk * p.ks[1];
    const __bf16* y2 = C::KV_SIDE ? p.dO + ((int64_t)b * p.H_q + hq) * p.L_q * C::DV : p.V + b * p.vs[0] + hk * p.vs[1];
    const int64_t s1 = C::KV_SIDE ? p.qs[2] : p.ks[2], s2 = C::KV_SIDE ? (int64_t)C::DV : p.vs[2];
    const uint32_t base = lds0 + stage * C::STAGE_BYTES;
#pragma unroll
    for (int i = 0; i < C::TILE * C::CPR1 / 64 / C::WAVES; ++i) {
      const int nb = wave + i * C::WAVES, pos = nb * 64 + lane;
      const int r = pos / C::CPR1, pc = pos % C::CPR1;
      int row = r0 + r;
      row = row < L_oth ? row : L_oth - 1;
      const uint32_t goff = (uint32_t)(((int64_t)row * s1 + ((pc ^ bswz<C::CPR1>(r)) * 8)) * 2);
      dma16(y1, goff, base + nb * 1024);
    }
#pragma unroll
    for (int i = 0; i < C::TILE * C::CPR2 / 64 / C::WAVES; ++i) {
      const int nb = wave + i * C::WAVES, pos = nb * 64 + lane;
      const int r = pos / C::CPR2, pc = pos % C::CPR2;
      int row = r0 + r;
      row = row < L_oth ? row : L_oth - 1;
      const uint32_t goff = (uint32_t)(((int64_t)row * s2 + ((pc ^ bswz<C::CPR2>(r)) * 8)) * 2);
      dma16(y2, goff, base + C::Y1_BYTES + nb * 1024);
    }
    if constexpr (C::BIAS) {
      // The block of the bias tensor that this tile meets, rows = queries.  Query side: 128 rows x 128 bytes
      // (8 chunks), chunk slot c ^ ((row >> 1) & 7); key side: 64 rows x 256 bytes (16 chunks), slot
      // c ^ ((row & 3) << 2) (read back transposed, 4 rows x 64 bytes at a time).  Chunks that start beyond the
      // last key are redirected to the row's last chunk (rows are padded to 8 elements by contract).
      const __bf16* bb = p.bias + b * p.bs[0] + hq * p.bs[1];
      constexpr int CPRB = C::KV_SIDE ? 16 : 8;
      const int q0 = C::KV_SIDE ? r0 : own0, k0 = C::KV_SIDE ? own0 : r0;
      const int last = ((p.L_k - 1) >> 3) << 3;
#pragma unroll
      for (int i = 0; i < 16 / C::WAVES; ++i) {
        const int nb = wave + i * C::WAVES, pos = nb * 64 + lane;
        const int r = pos / CPRB, pc = pos % CPRB;
        const int c = C::KV_SIDE ? pc ^ ((r & 3) << 2) : pc ^ ((r >> 1) & 7);
        int row = q0 + r, col = k0 + 8 * c;
        row = row < p.L_q ? row : p.L_q - 1;
        col = col < p.L_k ? col : last;
        dma16(bb, (uint32_t)(((int64_t)row * p.bs[2] + col) * 2), bias0 + stage * C::BIAS_BYTES + nb * 1024);
      }
    }
  };
  // key side: the tile's row quantities, wave 0 -> (bias - lse) * log2(e), wave 1 -> delta.  The
  // values are requested when the tile's copy starts and only touched (converted, written to LDS)
  // after the work on the tile before it: nothing waits for memory in between.
  auto load_rowq = [&](int n) -> float {
    float v = 0.f;
    if constexpr (C::KV_SIDE && C::ROWS) {
      if (wave < 2 && lane < C::TILE) {
        const int hq = hk * p.g + n / nt;
        const int i = (t_first + n % nt) * C::TILE + lane;
        const int64_t r = ((int64_t)b * p.H_q + hq) * p.L_q + i;
        const float* src = wave == 0 ? p.lse : p.delta;
        v = wave == 0 ? (C::ABS ? 0.f : -INFINITY) : 0.f;
        if (i < p.L_q) v = src[r];
      }
    }
    return v;
  };
  auto store_rowq = [&](float v, int stage) {
    if constexpr (C::KV_SIDE && C::ROWS) {
      if (wave < 2 && lane < C::TILE) {
        if (wave == 0) v = C::ABS ? fast_rcp(fmaxf(fabsf(v), 1.f)) : v == -INFINITY ? -INFINITY : p.b2 - v * 1.4426950408889634f;
        *reinterpret_cast<__attribute__((address_space(3))) float*>(
            (lds_char*)(uintptr_t)(rows0 + stage * C::ROW_BYTES + wave * C::TILE * 4 + lane * 4)) = v;
      }
    }
  };

  f32x16 g[C::DB], g2[C::HAS2 ? C::DB2 : 1];
#pragma unroll
  for (int d = 0; d < C::DB; ++d) g[d] = zero16();
#pragma unroll
  for (int d = 0; d < C::DB2; ++d) g2[d] = zero16();

  // Per-lane LDS addresses of the fragments in stage 0, sub-tile 0, step 0; stage, sub-tile and
  // 16-row step add compile-time constants (the swizzle only depends on the row modulo 16).
  //   ar1[t], ar2[t]: row fragment of contraction step t, row lane % 32 (A operand of S / dP);
  //   atl[k], ath[k]: the two transposing reads of 32-column block k, rows 4*half + i/4 (+8).
  constexpr int RBT = C::RB1;  // row bytes of the Y1 tile, read transposed for dQ^T / dK^T
  const int f1 = bswz<C::CPR1>(ln), f2 = bswz<C::CPR2>(ln);
  const int li = lane & 15, blk = (lane >> 4) & 1;
  const int trow = 4 * half + (li >> 2), tcl = 2 * blk + ((li & 3) >> 1);
  const int flo = bswz<RBT / 16>(trow), fhi = bswz<RBT / 16>(trow + 8);
  const uint32_t rb1 = lds0 + ln * C::RB1, rb2 = lds0 + C::Y1_BYTES + ln * C::RB2;
  const uint32_t tbl = lds0 + (li & 1) * 8 + trow * RBT, tbh = tbl + 8 * RBT;
  auto a_r1 = [&](int t) { return rb1 + (((2 * t + half) ^ f1) << 4); };
  auto a_r2 = [&](int t) { return rb2 + (((2 * t + half) ^ f2) << 4); };
  auto a_tl = [&](int k) { return tbl + (((4 * k + tcl) ^ flo) << 4); };
  auto a_th = [&](int k) { return tbh + (((4 * k + tcl) ^ fhi) << 4); };
  uint32_t ar1[C::T1], ar2[C::T2], atl[C::DB], ath[C::DB];
  uint32_t atl2[C::HAS2 ? C::DB2 : 1], ath2[C::HAS2 ? C::DB2 : 1];  // key side: the same for the Y2 tile
  if constexpr (C::HAS2) {
    const int glo = bswz<C::CPR2>(trow), ghi = bswz<C::CPR2>(trow + 8);
    const uint32_t t2 = lds0 + C::Y1_BYTES + (li & 1) * 8 + trow * C::RB2;
#pragma unroll
    for (int k = 0; k < C::DB2; ++k) {
      atl2[k] = t2 + (((4 * k + tcl) ^ glo) << 4);
      ath2[k] = t2 + 8 * C::RB2 + (((4 * k + tcl) ^ ghi) << 4);
    }
  }
  {
#pragma unroll
    for (int t = 0; t < C::T1; ++t) ar1[t] = a_r1(t);
#pragma unroll
    for (int t = 0; t < C::T2; ++t) ar2[t] = a_r2(t);
#pragma unroll
    for (int k = 0; k < C::DB; ++k) {
      atl[k] = a_tl(k);
      ath[k] = a_th(k);
    }
  }

  // One 32-row sub-tile of the other side (STAGE, SUB: compile-time LDS position; o0: its first row).
  auto subtile = [&](auto stagec, auto subc, int o0) {
    constexpr int STAGE = decltype(stagec)::value, SUB = decltype(subc)::value;
    // anything visible to this wave's rows?  everything?
    bool any = o0 < L_oth, full = o0 + 31 < L_oth;
    if constexpr (C::CAUSAL) {
      const int wd = p.window;
      if constexpr (C::KV_SIDE) {  // own = keys j, other = queries i: visible iff i + off - window < j <= i + off
        any = any && ow0 <= o0 + 31 + off && o0 + off - wd < ow0 + 31;
        full = full && ow0 + 31 <= o0 + off && o0 + 31 + off - wd < ow0;
      } else {                     // own = queries i, other = keys j
        any = any && o0 <= ow0 + 31 + off && ow0 + off - wd < o0 + 31;
        full = full && o0 + 31 <= ow0 + off && ow0 + 31 + off - wd < o0;
      }
    }
    if (!any) return;
    constexpr uint32_t kRow1 = STAGE * C::STAGE_BYTES + SUB * 32 * C::RB1, kRow2 = STAGE * C::STAGE_BYTES + SUB * 32 * C::RB2;
    // key side: the row quantities of the 16 rows this lane sees, requested ahead of the MFMAs that
    // hide their latency (register r is other-side row o0 + 8*(r/4) + 4*half + (r%4))
    constexpr uint32_t kRq = 2 * C::STAGE_BYTES + STAGE * C::ROW_BYTES + SUB * 32 * 4;
    constexpr bool ROWQ = C::ROWS && C::KV_SIDE;
    f32x4 nl4[4], dl4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      nl4[q] = f32x4{nl_own, nl_own, nl_own, nl_own};
      dl4[q] = f32x4{dl_own, dl_own, dl_own, dl_own};
      if constexpr (ROWQ) nl4[q] = lds_read16(lds0 + kRq + (8 * q + 4 * half) * 4);
    }
    if constexpr (ROWQ) sched_fence();
    f32x16 s = zero16(), dp = zero16();
    // the fragments of the accumulation step: tr[t][k], k < DB from Y1, the rest (key side) from Y2
    constexpr uint32_t kT = STAGE * C::STAGE_BYTES + SUB * 32 * RBT, kT2 = STAGE * C::STAGE_BYTES + SUB * 32 * C::RB2;
    auto read_acc = [&](int t, int k) {
      if constexpr (C::HAS2) {
        if (k >= C::DB) return read_tr_frag(atl2[k - C::DB] + kT2 + t * 16 * C::RB2, ath2[k - C::DB] + kT2 + t * 16 * C::RB2);
      }
      return read_tr_frag(atl[k < C::DB ? k : 0] + kT + t * 16 * RBT, ath[k < C::DB ? k : 0] + kT + t * 16 * RBT);
    };
    bf16x8 tr[2][C::BATCH ? C::DB + C::DB2 : 1];
    if constexpr (C::BATCH) {
      // One wave per SIMD: nothing else hides the LDS latency, so all fragments of a step are
      // requested before its first MFMA, and those of the accumulation step before the elementwise
      // step (the fences keep the compiler from sinking the reads back to their uses).
      bf16x8 a1[C::T1], a2[C::T2];
#pragma unroll
      for (int t = 0; t < C::T1; ++t) a1[t] = read_k_frag(ar1[t] + kRow1);
#pragma unroll
      for (int t = 0; t < C::T2; ++t) a2[t] = read_k_frag(ar2[t] + kRow2);
      sched_fence();
#pragma unroll
      for (int t = 0; t < C::T1; ++t) s = mfma(a1[t], xb1[t], s);
#pragma unroll
      for (int t = 0; t < C::T2; ++t) dp = mfma(a2[t], xb2[t], dp);
      sched_fence();
#pragma unroll
      for (int k = 0; k < C::DB + C::DB2; ++k) tr[0][k] = read_acc(0, k);
      sched_fence();
    } else {
#pragma unroll
      for (int t = 0; t < C::T1; ++t) s = mfma(read_k_frag(ar1[t] + kRow1), xb1[t], s);
#pragma unroll
      for (int t = 0; t < C::T2; ++t) dp = mfma(read_k_frag(ar2[t] + kRow2), xb2[t], dp);
    }
    float x[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = __builtin_fmaf(s[r], p.c2, C::NORM == NORM_SOFTMAX ? nl4[r / 4][r % 4] : p.b2);
    if constexpr (C::BIAS) {
      // register r = 4 q4 + e is (query, key) = (own row, key 8 q4 + 4 half + e of the sub-tile) on the query side,
      // (query 8 q4 + 4 half + e of the sub-tile, own key) on the key side
      const uint32_t bt = bias0 + STAGE * C::BIAS_BYTES;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        uint32_t lo, hi;
        if constexpr (C::KV_SIDE) {
          const int row = 32 * SUB + 8 * q4 + 4 * half + ((lane & 15) >> 2);   // the row this lane addresses
          const int cl = 4 * wave + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);  // chunk of its 4 columns
          const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)(
              bt + row * 256 + ((cl ^ ((row & 3) << 2)) << 4) + (lane & 1) * 8));
          const u32x2 w2 = __builtin_bit_cast(u32x2, v);
          lo = w2[0];
          hi = w2[1];
        } else {
          const int row = 32 * wave + ln;
          const u32x2 w2 = *reinterpret_cast<__attribute__((address_space(3))) const u32x2*>(
              (lds_char*)(uintptr_t)(bt + row * 128 + (((4 * SUB + q4) ^ ((row >> 1) & 7)) << 4) + 8 * half));
          lo = w2[0];
          hi = w2[1];
        }
        x[4 * q4 + 0] += __builtin_bit_cast(float, lo << 16) * p.bunit;
        x[4 * q4 + 1] += __builtin_bit_cast(float, lo & 0xffff0000u) * p.bunit;
        x[4 * q4 + 2] += __builtin_bit_cast(float, hi << 16) * p.bunit;
        x[4 * q4 + 3] += __builtin_bit_cast(float, hi & 0xffff0000u) * p.bunit;
      }
    }
    // abs-sum family: distance to the diagonal of register 0's entry, for the decay factor
    const float dist0 = (float)(C::KV_SIDE ? o0 + off - own + 4 * half : own + off - o0 - 4 * half);
    float f[C::LIN ? 16 : 1];  // decay factors
    if (!full) {  // a hidden entry gets the exponent (or the factors) that make its weight exactly 0
      sched_fence();  // (keeps this a branch: most sub-tiles skip it)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int oth = o0 + key_offset(r) + 4 * half;
        bool vis = oth < L_oth;
        if constexpr (C::CAUSAL)
          vis = vis && (C::KV_SIDE ? own <= oth + off && oth + off - p.window < own : oth <= own + off && own + off - p.window < oth);
        x[r] = vis ? x[r] : C::LIN ? 0.f : -INFINITY;
        if constexpr (C::LIN) {  // (visible entries have a distance >= 0)
          const float dist = dist0 + (C::KV_SIDE ? 1.f : -1.f) * (float)key_offset(r);
          f[r] = vis ? fast_exp2(lg * fmaxf(dist, 0.f)) : kHiddenFactor;
        }
      }
      sched_fence();
    } else if constexpr (C::LIN) {
      const float near = fast_exp2(lg * (C::KV_SIDE ? dist0 : dist0 - 27.f));
#pragma unroll
      for (int r = 0; r < 16; ++r) f[r] = near * dec_q[r / 4] * dec_e[r % 4];
      sched_fence();
    }
    float w[16], w2[C::HAS2 ? 16 : 1];  // the weight (dV) or the score gradient (dQ, dK); key side: both
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if constexpr (ROWQ)
        if (r % 4 == 0) dl4[r / 4] = lds_read16(lds0 + kRq + C::TILE * 4 + (8 * (r / 4) + 4 * half) * 4);
      float pv;
      if constexpr (C::NORM == NORM_SOFTMAX) {
        pv = fast_exp2(x[r]);
        if constexpr (C::HAS2) w2[r] = pv;
        pv = pv * (dp[r] - dl4[r / 4][r % 4]);
      } else if constexpr (C::NORM == NORM_SIGMOID) {
        pv = fast_rcp(1.f + fast_exp2(-x[r]));
        if constexpr (C::HAS2) w2[r] = pv;
        pv = dp[r] * pv * (1.f - pv);
      } else if constexpr (C::LIN) {
        const float dl = dl4[r / 4][r % 4];
        f[r] *= nl4[r / 4][r % 4];
        const float pw = x[r] * f[r];
        if constexpr (C::HAS2) w2[r] = pw;
        // g * delta: delta with its sign flipped where S' < 0 (abs-sum), or delta already signed by the row sum
        const float corr = C::NORM == NORM_ABSSUM
                               ? __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, dl) ^ (__builtin_bit_cast(uint32_t, pw) & 0x80000000u))
                               : dl;
        pv = (dp[r] - corr) * f[r];
      } else if constexpr (C::NORM == BWD_NORM_NONE_RELU) {  // P = max(x, 0); a hidden entry has x = -inf
        if constexpr (C::HAS2) w2[r] = fmaxf(x[r], 0.f);
        pv = x[r] > 0.f ? dp[r] : 0.f;
      }
      w[r] = pv;
    }
    if constexpr (C::LIN)
      if (!full) {  // a hidden entry's gradient is 0 whatever dP is (the product of a factor 0 with an infinite one is NaN)
        sched_fence();
#pragma unroll
        for (int r = 0; r < 16; ++r) w[r] = factor_hidden(f[r]) ? 0.f : w[r];
        sched_fence();
      }
    if constexpr (C::BIAS && !C::KV_SIDE) {
      // the bias enters S' with slope 1: its gradient is dS' itself, 4 x 4 consecutive keys of the lane's own row
      if (p.dbias != nullptr && own < p.L_q) {
        __bf16* drow = p.dbias + (((int64_t)b * p.H_q + ho) * p.L_q + own) * p.dbias_ld + o0 + 4 * half;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          if (o0 + 8 * q4 + 4 * half < p.L_k) {  // (a group across the last key writes into the row's padding)
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (__bf16)w[4 * q4 + e];
            *reinterpret_cast<bf16x4*>(drow + 8 * q4) = v;
          }
      }
    }
    if constexpr (C::BATCH) {
      sched_fence();
#pragma unroll
      for (int k = 0; k < C::DB + C::DB2; ++k) tr[1][k] = read_acc(1, k);
      sched_fence();
    }
    // G^T += Y^T W: per 16-row step t, the DB blocks of Y1^T (dQ^T, dK^T), then (key side) the DB2 blocks of Y2^T
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const bf16x8 wb = pack8(w, t);
#pragma unroll
      for (int k = 0; k < C::DB; ++k) g[k] = mfma(C::BATCH ? tr[t][C::BATCH ? k : 0] : read_acc(t, k), wb, g[k]);
      if constexpr (C::HAS2) {
        const bf16x8 pb = pack8(w2, t);
#pragma unroll
        for (int k = 0; k < C::DB2; ++k) g2[k] = mfma(C::BATCH ? tr[t][C::BATCH ? C::DB + k : 0] : read_acc(t, C::DB + k), pb, g2[k]);
      }
    }
  };
  // Tile n: wait for it, start the copy of tile n + 1 into the other stage, work on it.
  auto tile = [&](auto stagec, int n) {
    constexpr int STAGE = decltype(stagec)::value;
    // tile n has landed, and every wave is done with the stage that tile n + 1 goes to
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    float rowq_next = 0.f;
    if (n + 1 < total) {
      issue_tile(n + 1, STAGE ^ 1);
      rowq_next = load_rowq(n + 1);
    }
    const int r0 = (t_first + (C::KV_SIDE ? n % nt : n)) * C::TILE;
    if constexpr (C::KV_SIDE && C::LIN)
      if (n % nt == 0) set_decay(hk * p.g + n / nt);
    subtile(stagec, std::integral_constant<int, 0>{}, r0);
    subtile(stagec, std::integral_constant<int, 1>{}, r0 + 32);
    if (n + 1 < total) store_rowq(rowq_next, STAGE ^ 1);
  };

  if (total > 0) {
    issue_tile(0, 0);
    store_rowq(load_rowq(0), 0);
  }
  // Everything loaded so far is consumed here once.  Otherwise the compiler, which must assume at
  // the loop's entry that those loads may still be in flight, waits for vmcnt to drain in front of
  // the MFMAs inside the loop -- and vmcnt also counts the tile copies, so every tile would wait for
  // the copy of the next one instead of running beside it.
#pragma unroll
  for (int t = 0; t < C::T1; ++t) asm volatile("" ::"v"(xb1[t]));
#pragma unroll
  for (int t = 0; t < C::T2; ++t) asm volatile("" ::"v"(xb2[t]));
  asm volatile("" ::"v"(nl_own), "v"(dl_own));
  for (int n = 0; n < total; n += 2) {
    tile(std::integral_constant<int, 0>{}, n);
    if (n + 1 < total) tile(std::integral_constant<int, 1>{}, n + 1);
  }

  // ---- results: register r of block db is column own, row d = 32 db + 8 (r/4) + 4 half + r%4 ----
  if (own < L_own) {
    constexpr int D = C::DQK;
    float* o = (C::KV_SIDE ? p.dK + ((int64_t)b * p.H_kv + hk) * p.L_k * D : p.dQ + ((int64_t)b * p.H_q + ho) * p.L_q * D) +
               (int64_t)own * D;
    const float f = p.scale;
#pragma unroll
    for (int db = 0; db < C::DB; ++db)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4*>(o + 32 * db + 8 * q + 4 * half) =
            f32x4{g[db][4 * q] * f, g[db][4 * q + 1] * f, g[db][4 * q + 2] * f, g[db][4 * q + 3] * f};
    if constexpr (C::HAS2) {
      float* o2 = p.dV + (((int64_t)b * p.H_kv + hk) * p.L_k + own) * C::DV;
#pragma unroll
      for (int db = 0; db < C::DB2; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<f32x4*>(o2 + 32 * db + 8 * q + 4 * half) =
              f32x4{g2[db][4 * q], g2[db][4 * q + 1], g2[db][4 * q + 2], g2[db][4 * q + 3]};
    }
  }
}

// ---- two wavefronts per 32 own rows -------------------------------------------------------------------------------
// Role 0 (wavefronts 0..3) keeps X1 and X2, computes S, dP, the weights P and their gradients dS', and hands P (key side)
// and dS' on in LDS, in bfloat16 and in the order in which the other role's products take them.  Role 1 (wavefronts 4..7, on
// the same SIMDs) keeps the accumulators and does nothing but products: dV and dK, or dQ.  The products split evenly on the
// key side, D_qk + D_v of each.  Role 1 is a tile of 32 rows behind, so one barrier per tile hands over P and dS', the
// tiles that have landed and the stages that are free.  Role 1 starts every tile with products while role 0 computes S, and
// role 0's exponentials stand between its products of dP.
//
// Measured against a split in which role 0 computed S, the weights and dV and role 1 dP, dS' (from 32-bit factors that role 0
// handed on) and dK / dQ, us, key side + query side: 1 x 128 heads x 8192 192/128 causal softmax 5240 + 4160 -> 4980 + 3860, 8 x 12 x
// 4096 128/256 1265 + 850 -> 1200 + 795, abs-sum with decay 192/128 1215 + 990 -> 1120 + 857; key side of 128/128
// 4 x 32/8 x 2048 300 -> 285.  There role 1 waited for eight LDS reads behind every barrier and then ran its vector work, both
// in front of its products: 2430 clocks per tile of 1280 clocks of products, now 2020.  What bounds it now is power: the
// same kernels on inputs of zeros take 4030 + 3015 us (the first split 4500 + 3575), the clock falls from 2.06 to 1.91 GHz as the
// matrix units' share of the cycles goes from 0.48 and 0.49 to 0.54 and 0.59.  Left out for timing, of the 192/128 time: the copies 6-9 %,
// the row fragments 3 %, the transposed ones 5 %, the row quantities 1-2 %, the hand-over 3 %, the exponentials 5 %, all of them 22 %.
// Deeper rings, more products in front of the weights, raised wave priority: no difference.  The query side's copies all
// go with role 1, which has less to do there (role 0 or both: 2 % more).  Against two workgroups per CU where those
// fit (64/64; 128/128 query side, 4 x 32/8 x 2048 212) the pair takes longer (128/128 query side 250): the choice in bwd_launch.hpp.
template <int DQK_, int DV_, int NORM_, bool CAUSAL_, int OUT_, bool BIAS_ = false>
struct BwdPairCfg {
  static constexpr bool BIAS = BIAS_;
  static constexpr int DQK = DQK_, DV = DV_, NORM = NORM_, OUT = OUT_;
  static constexpr bool CAUSAL = CAUSAL_, KV_SIDE = OUT_ == BWD_DKV;
  static constexpr int WAVES = 8, THREADS = 512, OWN = 128, TILE = 32;
  static constexpr bool PAIR = true, OCC2 = false;
  static constexpr int T1 = DQK / 16, T2 = DV / 16, DB = DQK / 32, DB2 = KV_SIDE ? DV / 32 : 0;
  static constexpr bool ABS = NORM == NORM_ABSSUM || NORM == NORM_ABS_OF_SUM;
  static constexpr bool ROWS = NORM == NORM_SOFTMAX || ABS;
  static constexpr bool LIN = ABS || NORM == NORM_NONE;
  static constexpr bool ROWQ = ROWS && KV_SIDE;
  static constexpr int RB1 = DQK * 2, RB2 = DV * 2, CPR1 = DQK / 8, CPR2 = DV / 8;
  static constexpr int Y1_BYTES = TILE * RB1, Y2_BYTES = TILE * RB2, BIAS_BYTES = BIAS_ ? 8192 : 0;
  static constexpr int STAGE_BYTES = Y1_BYTES + Y2_BYTES + BIAS_BYTES;
  static constexpr int ROW_BYTES = ROWQ ? 512 : 0;  // per stage: [64] statistic, [64] delta (32 of each are used)
  static constexpr int STAGES = 5 * (STAGE_BYTES + ROW_BYTES) + 2 * 4 * 4096 <= 160 * 1024 ? 5 : 4, LOOK = STAGES - 2;
  static constexpr int ROWS0 = STAGES * STAGE_BYTES, E0 = ROWS0 + STAGES * ROW_BYTES, E_PAIR = KV_SIDE ? 4096 : 2048, E_BYTES = 4 * E_PAIR;
  static constexpr int LDS_BYTES = E0 + 2 * E_BYTES;
  static_assert(E_PAIR >= 2048, "a block of results takes 2 KB of either buffer");
  // copies: groups of four 1 KB blocks, group q by the wavefronts of role q % 2, or all by one role
  static constexpr int G1 = DQK / 64, G2 = DV / 64, GB = BIAS_ ? 2 : 0, GROUPS = G1 + G2 + GB;
  static constexpr int COPIER = KV_SIDE ? (DV == 256 && !LIN ? 0 : 2) : 1;  // 0, 1: that role; 2: both in turn
  // a lane's offsets of a short last tile are formed where they are used, in a branch, instead of being held in registers
  static constexpr bool TAIL_BRANCH = KV_SIDE && DV == 256 && LIN;
  // groups after which a lane's swizzle repeats (16 or 32 rows)
  static constexpr int copy_period(int cpr) { return cpr == 24 ? 3 : cpr == 32 ? 2 : 1; }
  // swizzle periods of the fragment addresses (in fragments): beyond them an address repeats at a fixed distance
  static constexpr int PR1 = CPR1 % 16 == 0 ? 8 : 4, PR2 = CPR2 % 16 == 0 ? 8 : 4;
  static constexpr int PK1 = CPR1 % 16 == 0 ? 4 : 2, PK2 = CPR2 % 16 == 0 ? 4 : 2;
  static_assert(LDS_BYTES <= 160 * 1024, "the workgroups of a CU must fit LDS");
};

// 64 lanes x 4 bytes from base + byte_off (per lane) to LDS bytes [lds_addr, lds_addr + 256)
__device__ __forceinline__ void dma4(const void* base_uniform, uint32_t byte_off, uint32_t lds_addr_uniform) {
  base_uniform = uniform_ptr(base_uniform);
  lds_addr_uniform = __builtin_amdgcn_readfirstlane(lds_addr_uniform);
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dword %1, %2"
      :
      : "s"(lds_addr_uniform), "v"(byte_off), "s"(base_uniform)
      : "memory", "m0");
}
__device__ __forceinline__ float lds_read4(uint32_t addr) {
  return *reinterpret_cast<__attribute__((address_space(3))) const float*>((lds_char*)(uintptr_t)addr);
}
__device__ __forceinline__ void lds_store4(uint32_t addr, float v) {
  *reinterpret_cast<__attribute__((address_space(3))) float*>((lds_char*)(uintptr_t)addr) = v;
}
__device__ __forceinline__ void lds_store16(uint32_t addr, u32x4 v) {
  *reinterpret_cast<__attribute__((address_space(3))) u32x4*>((lds_char*)(uintptr_t)addr) = v;
}

template <class C>
__device__ __forceinline__ void bwd_pair_walk(const BwdParams& p, const DecayTable& dt, int block, uint32_t lds0) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w4 = wave & 3;
  const int ln = lane & 31, half = lane >> 5;
  const int off = p.L_k - p.L_q;
  const int L_own = C::KV_SIDE ? p.L_k : p.L_q, L_oth = C::KV_SIDE ? p.L_q : p.L_k;

  const int n_own_tiles = (L_own + C::OWN - 1) / C::OWN;
  int group, item;
  if (!place_in_group(block, p.B * p.H_kv, C::KV_SIDE ? n_own_tiles : n_own_tiles * p.g, p.together[C::KV_SIDE ? 1 : 0], p.cut, group, item)) return;
  const int b = group / p.H_kv, hk = group % p.H_kv;
  const int ot = C::KV_SIDE ? item : n_own_tiles - 1 - item / p.g;
  const int ho = C::KV_SIDE ? hk : hk * p.g + item % p.g;  // ho: k/v head (key side) or q head (query side)
  const int own0 = ot * C::OWN, ow0 = own0 + w4 * 32;
  const int own = ow0 + ln;
  const int own_c = own < L_own ? own : L_own - 1;

  // ---- the walk over the other side, in tiles of 32 rows ----
  int t_first = 0, t_end = (L_oth + C::TILE - 1) / C::TILE;
  if constexpr (C::CAUSAL) {
    if constexpr (C::KV_SIDE) {
      const int i_first = own0 - off;  // first query that sees key own0
      t_first = i_first > 0 ? i_first / C::TILE : 0;
      if (t_first > t_end) t_first = t_end;
      const int i_last = own0 + C::OWN - 1 - off + p.window - 1;  // last query whose window holds a key here
      const int e = i_last < 0 ? 0 : i_last / C::TILE + 1;
      if (e < t_end) t_end = e;
      if (t_end < t_first) t_end = t_first;
    } else {
      const int j_last = own0 + C::OWN - 1 + off;  // last key any row here may see
      const int e = j_last < 0 ? 0 : j_last / C::TILE + 1;
      if (e < t_end) t_end = e;
      const int j_first = own0 + off - p.window + 1;  // first key inside the window of row own0
      t_first = j_first > 0 ? j_first / C::TILE : 0;
      if (t_first > t_end) t_first = t_end;
    }
  }
  const int N = (t_end - t_first) * (C::KV_SIDE ? p.g : 1);
  struct Pos {  // a position of the walk: tile t of q head h
    int t, h;
  };
  auto advance = [&](Pos& q) {
    if (++q.t == t_end) {
      q.t = t_first;
      ++q.h;
    }
  };
  const int h_first = C::KV_SIDE ? hk * p.g : ho;

  const int li = lane & 15, blk = (lane >> 4) & 1;
  const int trow = 4 * half + (li >> 2), tcl = 2 * blk + ((li & 3) >> 1);

  auto walk = [&](auto rolec) {
    constexpr int ROLE = decltype(rolec)::value;  // 0: scores, weights and their gradients, 1: the sums dV, dK / dQ
    constexpr int NC = C::COPIER == 2 ? (C::GROUPS - ROLE + 1) / 2 : C::COPIER == ROLE ? C::GROUPS : 0;  // copies of a tile
    constexpr int NCQ = C::COPIER == 2 ? 2 : 1, Q0 = C::COPIER == 2 ? ROLE : 0;  // copy k is group k NCQ + Q0

    // ---- copies ----
    const int64_t s1 = C::KV_SIDE ? p.qs[2] : p.ks[2], s2 = C::KV_SIDE ? (int64_t)C::DV : p.vs[2];
    const int tail = (L_oth - 1) % C::TILE;  // the last tile's last row: rows past it repeat it
    constexpr int PER1 = C::copy_period(C::CPR1), PER2 = C::copy_period(C::CPR2);
    auto copy_offset = [&](auto cprc, int Q, int64_t stride, int last) {  // the lane's byte offset from the tile's first row, group Q
      constexpr int CPR = decltype(cprc)::value;
      const int pos = (4 * Q + w4) * 64 + lane, r = pos / CPR, c = (pos % CPR) ^ bswz<CPR>(r);
      return (uint32_t)((min(r, last) * stride + c * 8) * 2);
    };
    constexpr std::integral_constant<int, C::CPR1> cpr1{};
    constexpr std::integral_constant<int, C::CPR2> cpr2{};
    uint32_t co[NC > 0 ? NC : 1], co_tail[NC > 0 ? NC : 1], co1[PER1], co2[PER2];  // co: of copy k; co1, co2: TAIL_BRANCH
    static_for<0, NC>([&](auto kc) {
      constexpr int k = decltype(kc)::value, q = k * NCQ + Q0;
      if constexpr (q < C::G1) {
        co[k] = copy_offset(cpr1, q, s1, C::TILE);
        co_tail[k] = copy_offset(cpr1, q, s1, tail);
      } else if constexpr (q < C::G1 + C::G2) {
        co[k] = copy_offset(cpr2, q - C::G1, s2, C::TILE);
        co_tail[k] = copy_offset(cpr2, q - C::G1, s2, tail);
      }
    });
#pragma unroll
    for (int k = 0; k < PER1; ++k) co1[k] = copy_offset(cpr1, k, s1, C::TILE);
#pragma unroll
    for (int k = 0; k < PER2; ++k) co2[k] = copy_offset(cpr2, k, s2, C::TILE);
    // the copies' own position in the walk, with the addresses of its tile's first rows
    Pos ahead{t_first, h_first};
    const __bf16 *y1, *y2;
    auto head_start = [&]() {
      y1 = (C::KV_SIDE ? p.Q + b * p.qs[0] + ahead.h * p.qs[1] : p.K + b * p.ks[0] + hk * p.ks[1]) + (int64_t)t_first * C::TILE * s1;
      y2 = (C::KV_SIDE ? p.dO + ((int64_t)b * p.H_q + ahead.h) * p.L_q * C::DV : p.V + b * p.vs[0] + hk * p.vs[1]) + (int64_t)t_first * C::TILE * s2;
    };
    head_start();
    const int h_last = h_first + (C::KV_SIDE ? p.g : 1) - 1;
    auto advance_copies = [&]() {  // (past the end of the walk the last tile is copied again, to stages that nobody reads)
      if (ahead.t + 1 < t_end) {
        y1 += C::TILE * s1;
        y2 += C::TILE * s2;
        ++ahead.t;
      } else if (ahead.h < h_last) {
        ahead.t = t_first;
        ++ahead.h;
        head_start();
      }
    };
    // copy instruction k of this wavefront for the tile that the copies stand at
    auto issue = [&](auto stagec, auto kc) {
      constexpr int ST = decltype(stagec)::value, k = decltype(kc)::value, q = k * NCQ + Q0;
      const int r0 = ahead.t * C::TILE;
      const uint32_t base = lds0 + ST * C::STAGE_BYTES;
      if constexpr (q < C::G1 + C::G2) {
        constexpr bool FIRST = q < C::G1;
        constexpr int Q = FIRST ? q : q - C::G1, PER = FIRST ? PER1 : PER2, ROWS = PER * 256 / (FIRST ? C::CPR1 : C::CPR2);
        uint32_t o;
        const __bf16* y = FIRST ? y1 : y2;
        if constexpr (!C::TAIL_BRANCH) {
          o = r0 + C::TILE > L_oth ? co_tail[k] : co[k];
        } else if (r0 + C::TILE > L_oth) {
          asm volatile("" ::: "memory");  // (keeps this a branch, and what it computes out of the loop's registers)
          if constexpr (FIRST) o = copy_offset(cpr1, Q, s1, tail);
          else o = copy_offset(cpr2, Q, s2, tail);
        } else {
          o = FIRST ? co1[Q % PER1] : co2[Q % PER2];
          y += Q / PER * ROWS * (FIRST ? s1 : s2);
        }
        dma16(y, o, base + (FIRST ? 0 : C::Y1_BYTES) + (4 * Q + w4) * 1024);
      } else {
        // The block of the bias tensor that this tile meets, rows = queries.  Query side: 128 rows x 64 bytes
        // (4 chunks), chunk slot c ^ ((row >> 2) & 3); key side: 32 rows x 256 bytes (16 chunks), slot
        // c ^ ((row & 3) << 2) (read back transposed, 4 rows x 64 bytes at a time).  Chunks that start beyond the
        // last key are redirected to the row's last chunk (rows are padded to 8 elements by contract).
        constexpr int CPRB = C::KV_SIDE ? 16 : 4;
        const __bf16* bb = p.bias + b * p.bs[0] + ahead.h * p.bs[1];
        const int nb = 4 * (q - C::G1 - C::G2) + w4, pos = nb * 64 + lane, r = pos / CPRB, pc = pos % CPRB;
        const int c = C::KV_SIDE ? pc ^ ((r & 3) << 2) : pc ^ ((r >> 2) & 3);
        int row = (C::KV_SIDE ? r0 : own0) + r, col = (C::KV_SIDE ? own0 : r0) + 8 * c;
        row = row < p.L_q ? row : p.L_q - 1;
        col = col < p.L_k ? col : ((p.L_k - 1) >> 3) << 3;
        dma16(bb, (uint32_t)(((int64_t)row * p.bs[2] + col) * 2), base + C::Y1_BYTES + C::Y2_BYTES + nb * 1024);
      }
    };
    // key side: 32 row quantities of a tile (lanes 32..63 repeat the last row of the query head)
    auto issue_rows = [&](auto stagec) {
      if constexpr (C::ROWQ) {
        constexpr int ST = decltype(stagec)::value;
        if (NC > 0 && w4 == 0) {
          const int i = min(ahead.t * C::TILE + lane, p.L_q - 1);
          const int64_t row0 = ((int64_t)b * p.H_q + ahead.h) * p.L_q;
          const uint32_t rows = lds0 + C::ROWS0 + ST * C::ROW_BYTES;
          if constexpr (ROLE == 0 || C::COPIER == 1) dma4(p.lse + row0, (uint32_t)i * 4u, rows);
          if constexpr (ROLE == 1 || C::COPIER == 0) dma4(p.delta + row0, (uint32_t)i * 4u, rows + 256);
        }
      }
    };
    auto all_copies = [&](auto copyc) {
      static_for<0, NC>([&](auto kc) { issue(copyc, kc); });
    };
    // The copies of a tile go out one instruction at a time between the M products of this role: queued together they would
    // hold up every wavefront at the compute unit's memory pipe (64 bytes per clock).
    auto copies = [&](auto copyc, auto nc, auto mc) {
      if constexpr (NC == 0) return;
      constexpr int n = decltype(nc)::value, M = decltype(mc)::value, GAP = M / (NC + 1) > 0 ? M / (NC + 1) : 1;
      static_assert((NC - 1) * GAP < M, "a product for every copy");
      if constexpr (n % GAP == 0 && n / GAP < NC) issue(copyc, std::integral_constant<int, n / GAP>{});
    };

    // the two buffers of the hand-over in turn, per pair and buffer: dS' (2 KB), weights (key side, 2 KB)
    uint32_t e_lane = lds0 + C::E0 + w4 * C::E_PAIR + lane * 16, e_flip = C::E_BYTES;

    // anything of the tile visible to this wave's rows?  everything?
    auto visibility = [&](int o0, bool& any, bool& full) {
      any = o0 < L_oth, full = o0 + 31 < L_oth;
      if constexpr (C::CAUSAL) {
        const int wd = p.window;
        if constexpr (C::KV_SIDE) {  // own = keys j, other = queries i: visible iff i + off - window < j <= i + off
          any = any && ow0 <= o0 + 31 + off && o0 + off - wd < ow0 + 31;
          full = full && ow0 + 31 <= o0 + off && o0 + 31 + off - wd < ow0;
        } else {                     // own = queries i, other = keys j
          any = any && o0 <= ow0 + 31 + off && ow0 + off - wd < o0 + 31;
          full = full && o0 + 31 <= ow0 + off && ow0 + 31 + off - wd < o0;
        }
      }
    };
    Pos here{t_first, h_first};  // the tile this role works on

    // Iteration i of the walk: tiles i and i + 1 have landed (of this wave's copies only the youngest LOOK - 2 tiles'
    // may be in flight), dS' and the weights of tile i - 1 are written (of role 0's LDS operations only the reads of
    // prefetch() may be in flight), and every wave is done with tile i - 2, whose stage takes tile i + LOOK.  Role 0
    // works on tile i, role 1 on tile i - 1.
    constexpr int RING = 4;  // LDS reads in flight ahead of their MFMAs (8 or 10: no faster, the key side of 192/128 spills)
    auto convert_stat = [&](float v) {
      return C::ABS ? fast_rcp(fmaxf(fabsf(v), 1.f)) : v == -INFINITY ? -INFINITY : p.b2 - v * 1.4426950408889634f;
    };
    auto convert_rows = [&](auto stagec) {  // the tile's statistics in LDS, as they arrived, into what the weights need
      if constexpr (C::ROWQ && ROLE == 0) {
        if (w4 == 0) {
          const uint32_t a = lds0 + C::ROWS0 + decltype(stagec)::value * C::ROW_BYTES + lane * 4;
          lds_store4(a, convert_stat(lds_read4(a)));
        }
      }
    };
    auto enter = [&](auto stagec) {
      constexpr int ST = decltype(stagec)::value;
      if constexpr (NC > 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((C::LOOK - 2) * NC) : "memory");
      if constexpr (ROLE == 0) asm volatile("s_waitcnt lgkmcnt(%0)\n\ts_barrier" ::"n"(RING) : "memory");
      else asm volatile("s_barrier" ::: "memory");
      convert_rows(std::integral_constant<int, (ST + 1) % C::STAGES>{});
      issue_rows(std::integral_constant<int, (ST + C::LOOK) % C::STAGES>{});
    };
    auto next_tile = [&]() {
      advance_copies();
      advance(here);
      e_lane += e_flip;
      e_flip = 0u - e_flip;
    };
    auto first_copies = [&]() {
      if (N > 0)
        static_for<0, C::LOOK>([&](auto nc) {
          issue_rows(nc);
          all_copies(nc);
          advance_copies();
        });
    };
    constexpr std::integral_constant<int, 0> first{};
    auto first_tiles_landed = [&]() {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      convert_rows(first);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    auto all_tiles = [&](auto step) {
#pragma clang loop unroll(disable)
      for (int n = 0; n < N; n += C::STAGES)
        static_for<0, C::STAGES>([&](auto uc) {
          if (n + decltype(uc)::value < N) step(uc, n + decltype(uc)::value);
        });
    };

    if constexpr (ROLE == 0) {
      constexpr int T1 = C::T1, T2 = C::T2, M = T1 + T2;
      // ---- own operands: B fragments, straight from global memory ----
      const __bf16* x1 = C::KV_SIDE ? p.K + b * p.ks[0] + hk * p.ks[1] + (int64_t)own_c * p.ks[2]
                                    : p.Q + b * p.qs[0] + ho * p.qs[1] + (int64_t)own_c * p.qs[2];
      const __bf16* x2 = C::KV_SIDE ? p.V + b * p.vs[0] + hk * p.vs[1] + (int64_t)own_c * p.vs[2]
                                    : p.dO + (((int64_t)b * p.H_q + ho) * p.L_q + own_c) * C::DV;
      bf16x8 xb1[T1], xb2[T2];
#pragma unroll
      for (int t = 0; t < T1; ++t) xb1[t] = *reinterpret_cast<const bf16x8*>(x1 + (2 * t + half) * 8);
#pragma unroll
      for (int t = 0; t < T2; ++t) xb2[t] = *reinterpret_cast<const bf16x8*>(x2 + (2 * t + half) * 8);
      // query side: the row quantities of the lane's own row (the statistic is converted behind the first copies)
      constexpr bool OWN_ROW = !C::KV_SIDE && C::ROWS;
      float nl_own = OWN_ROW ? (C::ABS ? 0.f : -INFINITY) : C::LIN ? 1.f : -INFINITY, dl_own = 0.f;
      if constexpr (OWN_ROW) {
        if (own < p.L_q) {
          nl_own = p.lse[((int64_t)b * p.H_q + ho) * p.L_q + own];
          dl_own = p.delta[((int64_t)b * p.H_q + ho) * p.L_q + own];
        }
      }
      // row fragments (stage 0): those of X1's product, then those of X2's
      constexpr int NR1 = T1 < C::PR1 ? T1 : C::PR1, NR2 = T2 < C::PR2 ? T2 : C::PR2;
      uint32_t ar1[NR1], ar2[NR2];
#pragma unroll
      for (int t = 0; t < NR1; ++t) ar1[t] = lds0 + ln * C::RB1 + (((2 * t + half) ^ bswz<C::CPR1>(ln)) << 4);
#pragma unroll
      for (int t = 0; t < NR2; ++t) ar2[t] = lds0 + C::Y1_BYTES + ln * C::RB2 + (((2 * t + half) ^ bswz<C::CPR2>(ln)) << 4);
      auto row_frag = [&](auto stagec, int n) {
        constexpr int o = decltype(stagec)::value * C::STAGE_BYTES;
        if (n < T1) return read_k_frag(ar1[n % C::PR1] + o + (n / C::PR1) * (C::PR1 * 32));
        const int t = n - T1;
        return read_k_frag(ar2[t % C::PR2] + o + (t / C::PR2) * (C::PR2 * 32));
      };
      bf16x8 fr[RING];  // the ring: the next tile's first fragments are carried from one iteration to the next
      auto prefetch = [&](auto stagec) {
#pragma unroll
        for (int n = 0; n < RING; ++n) fr[n] = row_frag(stagec, n);
      };
      // Decay factors of a tile whose entries are all visible: one exponential per lane, for the register with the shortest
      // distance, times these (register r = 4 q + e is q * 8 + e rows further on the key side, nearer on the query side).
      float lg = 0.f, dec_q[C::LIN ? 4 : 1], dec_e[C::LIN ? 4 : 1];
      auto set_decay = [&](int h) {
        if constexpr (C::LIN) {
          lg = p.has_decay ? dt.log2_gamma[h] : 0.f;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            dec_q[k] = fast_exp2(lg * (C::KV_SIDE ? 8.f * k : 24.f - 8.f * k));
            dec_e[k] = fast_exp2(lg * (C::KV_SIDE ? 1.f * k : 3.f - k));
          }
        }
      };
      set_decay(h_first);

      auto scores = [&](auto stagec, int o0) {
        constexpr int ST = decltype(stagec)::value;
        constexpr std::integral_constant<int, (ST + C::LOOK) % C::STAGES> copyc{};
        bool any, full;
        visibility(o0, any, full);
        if (!any) {
          all_copies(copyc);
          return;
        }
        f32x4 nl4[4], dl4[4];
        auto read_rows = [&](f32x4 (&v)[4], float own_value, int o) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            v[q] = f32x4{own_value, own_value, own_value, own_value};
            if constexpr (C::ROWQ) v[q] = lds_read16(lds0 + C::ROWS0 + ST * C::ROW_BYTES + o + (8 * q + 4 * half) * 4);
          }
        };
        if constexpr (!C::LIN) read_rows(nl4, nl_own, 0);
        sched_fence();
        f32x16 s = zero16(), dp = zero16();
        auto product = [&](auto nc) {
          constexpr int n = decltype(nc)::value;
          if constexpr (n < T1) s = mfma(fr[n % RING], xb1[n < T1 ? n : 0], s);
          else dp = mfma(fr[n % RING], xb2[n < T1 ? 0 : n - T1], dp);
          if constexpr (n + RING < M) fr[n % RING] = row_frag(stagec, n + RING);
          sched_fence();
          copies(copyc, nc, std::integral_constant<int, M>{});
        };
        constexpr int AHEAD = 2;  // products of dP in front of the first use of S: they cover its latency
        static_for<0, T1 + AHEAD>(product);
        if constexpr (C::LIN) read_rows(nl4, nl_own, 0);  // (here: 16 registers less during the products)
        float x[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = __builtin_fmaf(s[r], p.c2, C::NORM == NORM_SOFTMAX ? nl4[r / 4][r % 4] : p.b2);
        if constexpr (C::BIAS) {
          // register r = 4 q4 + e is (query, key) = (own row, key 8 q4 + 4 half + e of the tile) on the query side,
          // (query 8 q4 + 4 half + e of the tile, own key) on the key side
          const uint32_t bt = lds0 + ST * C::STAGE_BYTES + C::Y1_BYTES + C::Y2_BYTES;
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            uint32_t lo, hi;
            if constexpr (C::KV_SIDE) {
              const int row = 8 * q4 + 4 * half + ((lane & 15) >> 2);               // the row this lane addresses
              const int cl = 4 * w4 + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);    // chunk of its 4 columns
              const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)(
                  bt + row * 256 + ((cl ^ ((row & 3) << 2)) << 4) + (lane & 1) * 8));
              const u32x2 w2 = __builtin_bit_cast(u32x2, v);
              lo = w2[0];
              hi = w2[1];
            } else {
              const int row = 32 * w4 + ln;
              const u32x2 w2 = *reinterpret_cast<__attribute__((address_space(3))) const u32x2*>(
                  (lds_char*)(uintptr_t)(bt + row * 64 + ((q4 ^ ((row >> 2) & 3)) << 4) + 8 * half));
              lo = w2[0];
              hi = w2[1];
            }
            x[4 * q4 + 0] += __builtin_bit_cast(float, lo << 16) * p.bunit;
            x[4 * q4 + 1] += __builtin_bit_cast(float, lo & 0xffff0000u) * p.bunit;
            x[4 * q4 + 2] += __builtin_bit_cast(float, hi << 16) * p.bunit;
            x[4 * q4 + 3] += __builtin_bit_cast(float, hi & 0xffff0000u) * p.bunit;
          }
        }
        // abs-sum family, no normalization: distance to the diagonal of register 0's entry, and what turns dP - delta into dS'
        const float dist0 = (float)(C::KV_SIDE ? o0 + off - own + 4 * half : own + off - o0 - 4 * half);
        float f[C::LIN ? 16 : 1];
        if (!full) {  // a hidden entry gets the exponent (or the factors) that make its weight exactly 0
          sched_fence();  // (keeps this a branch: most tiles skip it)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int oth = o0 + key_offset(r) + 4 * half;
            bool vis = oth < L_oth;
            if constexpr (C::CAUSAL)
              vis = vis && (C::KV_SIDE ? own <= oth + off && oth + off - p.window < own : oth <= own + off && own + off - p.window < oth);
            x[r] = vis ? x[r] : C::LIN ? 0.f : -INFINITY;
            if constexpr (C::LIN) {  // (visible entries have a distance >= 0)
              const float dist = dist0 + (C::KV_SIDE ? 1.f : -1.f) * (float)key_offset(r);
              f[r] = vis ? fast_exp2(lg * fmaxf(dist, 0.f)) : kHiddenFactor;
            }
          }
          sched_fence();
        } else if constexpr (C::LIN) {
          const float near = fast_exp2(lg * (C::KV_SIDE ? dist0 : dist0 - 27.f));
#pragma unroll
          for (int r = 0; r < 16; ++r) f[r] = near * dec_q[r / 4] * dec_e[r % 4];
          sched_fence();
        }
        // the weights, a few of them between every two products of dP
        float pv[16];
        auto weight = [&](int r) {
          if constexpr (C::NORM == NORM_SOFTMAX) {
            pv[r] = fast_exp2(x[r]);
          } else if constexpr (C::NORM == NORM_SIGMOID) {
            pv[r] = fast_rcp(1.f + fast_exp2(-x[r]));
          } else if constexpr (C::LIN) {
            f[r] *= nl4[r / 4][r % 4];
            pv[r] = x[r] * f[r];
          } else {  // no normalization with ReLU
            pv[r] = fmaxf(x[r], 0.f);
          }
        };
        static_for<T1 + AHEAD, M>([&](auto nc) {
          constexpr int k = decltype(nc)::value - T1 - AHEAD, K = T2 - AHEAD;
#pragma unroll
          for (int r = 16 * k / K; r < 16 * (k + 1) / K; ++r) weight(r);
          sched_fence();
          product(nc);
        });
        read_rows(dl4, dl_own, 256);
        if constexpr (C::KV_SIDE) {
#pragma unroll
          for (int t = 0; t < 2; ++t) lds_store16(e_lane + 2048 + t * 1024, __builtin_bit_cast(u32x4, pack8(pv, t)));
        }
        sched_fence();
        float w[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float dl = dl4[r / 4][r % 4], d = dp[r];
          if constexpr (C::NORM == NORM_SOFTMAX) {
            w[r] = pv[r] * (d - dl);
          } else if constexpr (C::NORM == NORM_SIGMOID) {
            w[r] = d * pv[r] * (1.f - pv[r]);
          } else if constexpr (C::LIN) {
            // g * delta: delta with its sign flipped where S' < 0 (abs-sum), or delta already signed by the row sum
            const float corr =
                C::NORM == NORM_ABSSUM
                    ? __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, dl) ^ (__builtin_bit_cast(uint32_t, pv[r]) & 0x80000000u))
                    : dl;
            w[r] = (d - corr) * f[r];
          } else {
            w[r] = pv[r] > 0.f ? d : 0.f;
          }
        }
        if constexpr (C::LIN)
          if (!full) {  // a hidden entry's gradient is 0 whatever dP is (the product of a factor 0 with an infinite one is NaN)
            sched_fence();
#pragma unroll
            for (int r = 0; r < 16; ++r) w[r] = factor_hidden(f[r]) ? 0.f : w[r];
            sched_fence();
          }
        if constexpr (C::BIAS && !C::KV_SIDE) {
          // the bias enters S' with slope 1: its gradient is dS' itself, 4 x 4 consecutive keys of the lane's own row
          if (p.dbias != nullptr && own < p.L_q) {
            __bf16* drow = p.dbias + (((int64_t)b * p.H_q + ho) * p.L_q + own) * p.dbias_ld + o0 + 4 * half;
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
              if (o0 + 8 * q4 + 4 * half < p.L_k) {  // (a group across the last key writes into the row's padding)
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (__bf16)w[4 * q4 + e];
                *reinterpret_cast<bf16x4*>(drow + 8 * q4) = v;
              }
          }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) lds_store16(e_lane + t * 1024, __builtin_bit_cast(u32x4, pack8(w, t)));
      };

      first_copies();
      // The own operands, requested in front of the first copies, are consumed here once: the compiler must not wait for them
      // inside the loop, where its count would wait for the copies too.
#pragma unroll
      for (int t = 0; t < T1; ++t) pin(xb1[t]);
#pragma unroll
      for (int t = 0; t < T2; ++t) pin(xb2[t]);
      pin(nl_own);
      pin(dl_own);
      if constexpr (OWN_ROW) nl_own = convert_stat(nl_own);
      if (N > 0) {
        first_tiles_landed();
        prefetch(first);
        sched_fence();
        all_tiles([&](auto stagec, int n) {  // iteration n on tile n
          constexpr std::integral_constant<int, (decltype(stagec)::value + 1) % C::STAGES> nextc{};
          enter(stagec);
          scores(stagec, here.t * C::TILE);
          next_tile();
          sched_fence();
          prefetch(nextc);
          sched_fence();
          if constexpr (C::LIN && C::KV_SIDE)
            if (here.t == t_first && n + 1 < N) set_decay(here.h);
        });
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // iteration N
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (no copy outlives the workgroup's LDS)
      }
    } else {
      constexpr int DB = C::DB, DB2 = C::DB2, NB = DB + DB2, NF = 2 * NB;
      static_assert(NF % RING == 0, "the ring runs on from tile to tile");
      f32x16 acc[NB];
#pragma unroll
      for (int d = 0; d < NB; ++d) acc[d] = zero16();
      // transposed fragments (stage 0): blocks of Y1 (dK, dQ), then (key side) of Y2 (dV)
      constexpr int NK1 = DB < C::PK1 ? DB : C::PK1, NK2 = DB2 < C::PK2 ? DB2 : C::PK2;
      uint32_t at1[NK1][2], at2[NK2 > 0 ? NK2 : 1][2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int k = 0; k < NK1; ++k)
          at1[k][h] = lds0 + (li & 1) * 8 + (trow + 8 * h) * C::RB1 + (((4 * k + tcl) ^ bswz<C::CPR1>(trow + 8 * h)) << 4);
#pragma unroll
        for (int k = 0; k < NK2; ++k)
          at2[k][h] = lds0 + C::Y1_BYTES + (li & 1) * 8 + (trow + 8 * h) * C::RB2 + (((4 * k + tcl) ^ bswz<C::CPR2>(trow + 8 * h)) << 4);
      }
      // fragment n of the sums: 16-row step n / NB, block n % NB
      auto acc_frag = [&](auto stagec, int n) {
        const int t = n / NB, k = n % NB;
        const uint32_t st = decltype(stagec)::value * C::STAGE_BYTES;
        if (k < DB) {
          const uint32_t o = st + t * 16 * C::RB1 + (k / C::PK1) * (C::PK1 * 64);
          return read_tr_frag(at1[k % C::PK1][0] + o, at1[k % C::PK1][1] + o);
        }
        const int k2 = k - DB;
        const uint32_t o = st + t * 16 * C::RB2 + (k2 / C::PK2) * (C::PK2 * 64);
        return read_tr_frag(at2[k2 % C::PK2][0] + o, at2[k2 % C::PK2][1] + o);
      };
      bf16x8 f[RING];  // the ring, carried from tile to tile
      auto prefetch = [&](auto stagec) {
#pragma unroll
        for (int n = 0; n < RING; ++n) f[n] = acc_frag(stagec, n);
      };
      // the sums over tile n (stage stagec); the ring goes on with the tile behind it (stage nextc)
      auto sums = [&](auto stagec, auto nextc, int o0) {
        constexpr int ST = decltype(stagec)::value;
        constexpr std::integral_constant<int, (ST + 1 + C::LOOK) % C::STAGES> copyc{};
        bool any, full;
        visibility(o0, any, full);
        if (!any) {
          all_copies(copyc);
          prefetch(nextc);
          return;
        }
        bf16x8 wb[2], pb[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          wb[t] = read_k_frag(e_lane + t * 1024);
          if constexpr (C::KV_SIDE) pb[t] = read_k_frag(e_lane + 2048 + t * 1024);
        }
        sched_fence();
        static_for<0, NF>([&](auto nc) {
          constexpr int n = decltype(nc)::value, k = n % NB, t = n / NB;
          acc[k] = mfma(f[n % RING], k < DB ? wb[t] : pb[t], acc[k]);
          if constexpr (n + RING < NF) f[n % RING] = acc_frag(stagec, n + RING);
          else f[n % RING] = acc_frag(nextc, n + RING - NF);
          sched_fence();
          copies(copyc, nc, std::integral_constant<int, NF>{});
        });
      };

      first_copies();
      if (N > 0) {
        first_tiles_landed();
        enter(first);  // iteration 0
        prefetch(first);
        all_copies(std::integral_constant<int, C::LOOK>{});
        advance_copies();
        all_tiles([&](auto stagec, int n) {  // iteration n + 1 on tile n
          constexpr std::integral_constant<int, (decltype(stagec)::value + 1) % C::STAGES> nextc{};
          enter(nextc);
          sums(stagec, nextc, here.t * C::TILE);
          next_tile();
        });
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // (no copy outlives the workgroup's LDS)
      }

      // ---- results: register r of block db is column own, row d = 32 db + 8 (r/4) + 4 half + r%4 ----
      // A block of 32 x 32 is turned around in the pair's hand-over buffers, which nobody reads any more (16-byte chunk k of row r at
      // k ^ (r % 8), the upper 16 rows in the second buffer): eight lanes then store 128 bytes of a row.  These stores are the end of a
      // workgroup, with nothing beside them.  Pieces of 16 bytes from 32 rows each instead, us: 8 x 64 heads causal, 192/128, x 200 142 -> 132,
      // x 256 190 -> 160, x 512 412 -> 355, window 256 409 -> 353, unmasked x 128 84 -> 68; 128/128 x 256 140 -> 125;
      // 1 x 128 x 4096 192/128 2439 -> 2398.
      const int row = lane >> 3, rows = L_own - ow0 - row;
      const uint32_t buf = lds0 + C::E0 + w4 * C::E_PAIR;
      const uint32_t put = buf + (ln >> 4) * C::E_BYTES + (ln & 15) * 128 + ((half ^ (ln & 7)) << 4);
      const uint32_t get = buf + row * 128 + (((lane & 7) ^ row) << 4);
      const int64_t row0 = (C::KV_SIDE ? ((int64_t)b * p.H_kv + hk) * p.L_k : ((int64_t)b * p.H_q + ho) * p.L_q) + ow0 + row;
      float* const o1 = (C::KV_SIDE ? p.dK : p.dQ) + row0 * C::DQK + 4 * (lane & 7);
      float* const o2 = p.dV + row0 * C::DV + 4 * (lane & 7);  // (key side)
      auto put_block = [&](auto dbc) {
        constexpr int db = decltype(dbc)::value;
        const float f = db < DB ? p.scale : 1.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = {acc[db][4 * q] * f, acc[db][4 * q + 1] * f, acc[db][4 * q + 2] * f, acc[db][4 * q + 3] * f};
          lds_store16(put ^ (32 * q), __builtin_bit_cast(u32x4, v));
        }
      };
      f32x4 v[2][4];
      auto get_block = [&](f32x4 (&v)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = lds_read16(get + (k & 1) * 1024 + (k >> 1) * C::E_BYTES);
        sched_fence();
      };
      put_block(first);
      get_block(v[0]);
      static_for<0, NB>([&](auto dbc) {  // (LDS works in order: block db + 1 goes in behind the reads of block db, while these are on their way)
        constexpr int db = decltype(dbc)::value;
        if constexpr (db + 1 < NB) {
          put_block(std::integral_constant<int, db + 1>{});
          sched_fence();
          get_block(v[(db + 1) % 2]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) pin(v[db % 2][k]);  // (the compiler would read each piece where it is stored, one behind the other)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (8 * k < rows)
            *reinterpret_cast<f32x4*>(db < DB ? o1 + 8 * k * C::DQK + 32 * db : o2 + 8 * k * C::DV + 32 * (db - DB)) = v[db % 2][k];
      });
    }
  };
  if (wave < 4) walk(std::integral_constant<int, 0>{});
  else walk(std::integral_constant<int, 1>{});
}

// ---- the kernels ----------------------------------------------------------------------------------------------------
template <class C>
__device__ __forceinline__ void bwd_walk(const BwdParams& p, const DecayTable& dt, int block, uint32_t lds0) {
  if constexpr (C::PAIR) bwd_pair_walk<C>(p, dt, block, lds0);
  else bwd_single_walk<C>(p, dt, block, lds0);
}
// wavefronts per SIMD that the registers are shared among
template <class C>
constexpr int bwd_waves_per_simd() { return C::PAIR || C::OCC2 ? 2 : 1; }

// One side.
template <class C>
__global__ __launch_bounds__(C::THREADS, bwd_waves_per_simd<C>()) void attn_bwd_kernel(const BwdParams p, const DecayTable dt) {
  __shared__ __attribute__((aligned(1024))) char smem[C::LDS_BYTES];
  bwd_walk<C>(p, dt, blockIdx.x, (uint32_t)(uintptr_t)((lds_char*)smem));
}

// Both sides, the key side's workgroups (K) first: they need nothing of each other, and the second one's workgroups go where the
// first one's leave the device idle.
template <class K, class Q>
struct BwdBoth {
  static constexpr int THREADS = K::THREADS > Q::THREADS ? K::THREADS : Q::THREADS;
  static constexpr int LDS_BYTES = K::LDS_BYTES > Q::LDS_BYTES ? K::LDS_BYTES : Q::LDS_BYTES;
  static constexpr int WAVES_PER_SIMD = THREADS == 512 || bwd_waves_per_simd<K>() + bwd_waves_per_simd<Q>() == 4 ? 2 : 1;
};
template <class K, class Q>
__global__ __launch_bounds__((BwdBoth<K, Q>::THREADS), (BwdBoth<K, Q>::WAVES_PER_SIMD))
void attn_bwd_both_kernel(const BwdParams p, const DecayTable dt, int key_blocks) {
  __shared__ __attribute__((aligned(1024))) char smem[BwdBoth<K, Q>::LDS_BYTES];
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_char*)smem);
  // (wavefronts beyond those of the walk end here: a barrier counts those that are left)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), block = (int)blockIdx.x;
  if (block < key_blocks) {
    if (wave < K::WAVES) bwd_walk<K>(p, dt, block, lds0);
  } else {
    if (wave < Q::WAVES) bwd_walk<Q>(p, dt, block - key_blocks, lds0);
  }
}

}  // namespace ae
