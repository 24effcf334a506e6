// Recurrent pattern with per-token gates, in one pass (paper Section 4.1, "Attention Patterns and Templates": K@V,
// then Q@h, iterated over a compressed state; "Examples of Attention variants": Mamba2's k_mod = k x gate and
// h_mod = h x decay x gate; Table 2: "Mamba2 SSM", "Gated Retention", "Retention Recurrent"; Section 4.2: chunk
// parallelism for the matrix units):
//     h_t = a_t h_{t-1} + (g_t k_t)^T v_t,     o_t = scale q_t h_t,        a_t = exp(log_decay_t) in (0, 1].
//
// One workgroup per (batch, value head) walks the sequence in chunks of 64 tokens with the state in registers
// (fp32 MFMA accumulators) from the first token to the last: Q, K, V are read once, O is written once, the state
// never touches memory (only h_in / h_out at the ends).  With b_i the sum of the log-decays from the chunk's first
// token to token i (b_i <= 0, decreasing), for token i of the chunk and H the state in front of the chunk:
//     o_i   = scale e^{b_i} q_i H  +  sum_{j <= i} scale e^{b_i - b_j} g_j (q_i . k_j) v_j
//     H_new = e^{b_last} H + sum_j (e^{b_last - b_j} g_j) k_j^T v_j
// Every exponent is <= 0: nothing overflows, nothing is divided by a decay.
//
// What bounds a walk is the latency chain of its chunks, and most of a chunk does not depend on the state: the weights of its
// 64 x 64 pairs and the gates.  So the work is split between two kinds of wavefronts, one of each on a SIMD, whose matrix and
// vector instructions overlap:
//   * state wavefronts, one per 32 value columns of a head: they keep the state slab [D_qk x 32] as D_qk / 32 accumulator tiles;
//     per chunk they read the state out for the 64 queries, add the weighted values, store the outputs and update the state;
//   * four helpers: three of them form the three 32 x 32 blocks of the chunk's weights that the causal order leaves (once
//     per chunk, not once per 32 value columns) and copy the tiles, the fourth makes the gates' sums and factors.  The scores
//     of a chunk are formed while the state wavefronts work on the chunk before, the weights while they read the state out.
// Two barriers per chunk: in front of the first one the state is read out and the weights are written, behind it the weights
// are used, the state is updated, and the next chunk's scores and gates are formed.
// All products are transposed so that a lane owns one column -- a
// query in S^T and O^T, a value column in H -- and the registers run over the contracted index:
//     S^T [keys x queries]   = K Q^T          A: K rows, B: Q rows (16-byte row pieces)
//     R^T [v x queries]      = H^T Q^T        A: the state accumulators themselves, packed to bf16 (lane = value
//                                                column, registers = d: an accumulator tile IS an A operand whose
//                                                contraction runs over its rows), B: Q rows, read like those of S^T
//     O^T += V^T P^T                          A: V through the transposing LDS read, B: the S^T accumulators,
//                                                weighted and packed (through LDS in the registers' own order)
//     H   += K^T (w . V)                      A: K through the transposing read, B: the same V fragments times
//                                                the per-token weights w_j = e^{b_last - b_j} g_j
// Row m of an accumulator tile of H is the column of K that lane m of the A operand reads.  The transposing read takes pieces
// of four columns from any address: pieces 1 and 2 of every 16 columns are exchanged, so that the eight registers a lane
// packs for the read-out are eight consecutive d, and a query fragment is one 16-byte read.
// The outputs of a chunk (32 queries x 32 columns per state wavefront and block) are turned around in LDS, where the chunk's
// queries were, and stored in whole 128-byte lines: as they stand, a store instruction would touch 32 rows of 32 bytes, and the
// compute unit's memory pipe takes about 60 clocks for each of those (16 for a kilobyte of whole lines).
// Q, K, V tiles arrive by LDS-DMA into a ring of three stages (chunk c is worked on, c + 1 is needed half a chunk later, c + 2
// is in flight).  Measured against the form without helpers, where every state wavefront formed the gates and, for its own 32
// columns, the weights (us, one card): 8 x 32 heads x 8192 tokens, 128/128, 592 -> 535 (5.0 TB/s: the memory's rate), 8 x 16 x 4096
// 64/64 119 -> 92, 1 x 4 x 300 128/128 21.0 -> 14.8, Mamba2 1 x 80 x 8192 (three launches) 137 -> 113, 8 x 80 x 2048 259 -> 180.
// The lanes' LDS addresses are formed chunk by chunk from one register for each kind of fragment and pinned there; left alone, the
// compiler carried 35 of them through the loop (64/64 144 registers, now 123; 1 x 32 x 2000 128/128 80 -> 73, 2 x 24/8 x 2000 128/64 74.5 -> 68.5).
// The same kernel serves the backward pass (other operands, a walk from the last token to the first,
// see GatedParams::reverse) and walks cut into segments (GatedParams::nseg).
#include <hip/hip_runtime.h>

#include "attn_bwd_kernel.hpp"  // bswz, read_tr_frag, lds_store4
#include "gated.hpp"

namespace ae {
namespace {

// HPW_: value heads per workgroup.  Heads of one q/k group (Mamba2: every head of a group reads the same B and C)
// can share the Q and K tiles, and the scores, of a workgroup: HPW_ consecutive heads, each with its own V tile, gates and state.
template <int DQK_, int DV_, int HPW_ = 1>
struct GCfg {
  static constexpr int DQK = DQK_, DV = DV_, HPW = HPW_, CH = 64;
  static constexpr int NB = DV / 32, SW = HPW * NB;  // state wavefronts: one per 32 value columns of a head
  static constexpr int WAVES = SW + 4, THREADS = 64 * WAVES;
  static constexpr int RBQ = DQK * 2, RBV = DV * 2, CPRQ = DQK / 8, CPRV = DV / 8;
  static constexpr int Q_BYTES = CH * RBQ, V_BYTES = CH * RBV;
  static constexpr int T = DQK / 16, DBQ = DQK / 32;
  // the gates' values of a head's chunk, in floats: b, u, s (see put_gates), two sets of w, the groups' references, two decays
  static constexpr int kB = 0, kU = 64, kS = 128, kW = 192, kRef = 320, kDec = 336, GATE_BYTES = 352 * 4;
  static constexpr int P_BYTES = 3 * 2048;  // per head: the chunk's weights, three blocks of 32 x 32 in bf16
  // 64/64, one head: two workgroups of six wavefronts per compute unit.  They were seen to share one only where a
  // SIMD has room for four wavefronts (as if both began on the same SIMD): 128 registers each.  With 144, for three, only one workgroup was resident, and 257 pairs took two rounds:
  // 9 x 32 heads x 1024 60 us, 42 now; 8 x 48 x 1024 62 / 47, its backward pass 229 / 184; 5 x 32 x 768 backward 74 / 55.
  // BOUND_THREADS: what the launch bound says, so that the compiler counts four wavefronts too.
  static constexpr bool SHARES_CU = DQK == 64 && DV == 64 && HPW == 1;
  static constexpr int WAVES_PER_SIMD = SHARES_CU ? 4 : 2, BOUND_THREADS = SHARES_CU ? 512 : THREADS;
};

// LDS layout: a stage holds the tiles Q (full walks only), K, V of every head
template <class C, bool STATE_ONLY>
struct GLayout {
  static constexpr int kK = STATE_ONLY ? 0 : C::Q_BYTES, kV = kK + C::Q_BYTES, STAGE_BYTES = kV + C::HPW * C::V_BYTES;
  // a state walk needs a chunk only when it updates with it and has the room: one more chunk in flight
  static constexpr int STAGES = STATE_ONLY ? 4 : 3;
  static constexpr int kP = STAGES * STAGE_BYTES, kGates = kP + (STATE_ONLY ? 0 : C::HPW * C::P_BYTES);
  // 4 KB per state wavefront to turn an output block around: the stage's queries, where they are large enough
  static constexpr bool kOutInQ = C::Q_BYTES >= C::SW * 4096;
  static constexpr int kOut = kGates + C::HPW * C::GATE_BYTES;
  static constexpr int LDS_BYTES = kOut + (STATE_ONLY || kOutInQ ? 0 : C::SW * 4096);
  static_assert(LDS_BYTES <= 160 * 1024 / (C::SHARES_CU ? 2 : 1), "tiles do not fit LDS");
};

// x of the lane that the control word selects, 0 where it selects none or the masks switch the lane off
template <int CTRL, int ROW_MASK, int BANK_MASK>
__device__ __forceinline__ float dpp_f(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, ROW_MASK, BANK_MASK, false));
}
__device__ __forceinline__ float lds_read4(uint32_t addr) {
  return *reinterpret_cast<__attribute__((address_space(3))) const float*>((lds_char*)(uintptr_t)addr);
}
// Workgroup barrier: this wavefront's LDS reads and writes are done (its copies in flight are not waited for).
__device__ __forceinline__ void chunk_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ---- fragments: the lane's part of their LDS addresses ----
// Transposed fragment: 32 columns (block k) of a tile of CPR chunks per row, rows 4 half + li / 4 (+ 8 for j = 1) of a 16-token
// step (lane = column, registers = rows in accumulator order); `piece`: which four columns of every 16.
template <int CPR>
__device__ __forceinline__ uint32_t tr_lane(int lane, int k, int j, int piece) {
  const int r = 4 * (lane >> 5) + ((lane & 15) >> 2) + 8 * j;
  return (uint32_t)((piece & 1) * 8 + r * (CPR * 16) + (((4 * k + 2 * ((lane >> 4) & 1) + (piece >> 1)) ^ bswz<CPR>(r)) << 4));
}
// pieces 1 and 2 of every 16 columns exchanged: the order that makes a lane's eight packed state registers consecutive rows d
__device__ __forceinline__ int swapped_piece(int lane) { return 2 * (lane & 1) + ((lane >> 1) & 1); }
// row fragment of Q or K for d-step 0 (d = 16 t + 8 half + {0..7} in step t), row lane % 32 of a 32-row block; in step t the
// address (tiles stand at multiples of 256 bytes) is that of step 0 with the bits of 32 t turned over
template <class C>
__device__ __forceinline__ uint32_t row_lane(int lane) {
  return (uint32_t)((lane & 31) * C::RBQ + (((lane >> 5) ^ bswz<C::CPRQ>(lane & 31)) << 4));
}

// ---- a state wavefront's share of a chunk ----
// O^T = H^T Q^T for both blocks of 32 queries (H rounded to bf16); in the same pass over the accumulators H takes the chunk's
// whole decay.  q: the lane's address of the first fragment of the queries.
template <class C>
__device__ __forceinline__ void read_out(f32x16 (&H)[C::DBQ], float dec, uint32_t q, f32x16& o0, f32x16& o1) {
  pin(q);
  o0 = zero16();
  o1 = zero16();
#pragma unroll
  for (int db = 0; db < C::DBQ; ++db) {
    bf16x8 hp[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float x = H[db][r];
      hp[r / 8][r % 8] = (__bf16)x;
      H[db][r] = x * dec;
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const uint32_t a = q ^ (32 * (2 * db + tt));
      o0 = mfma(hp[tt], read_k_frag(a), o0);
      o1 = mfma(hp[tt], read_k_frag(a + 32 * C::RBQ), o1);
    }
  }
}
// O^T += V^T P^T; weights at pb: block 0: queries 0-31 x keys 0-31, 1: 32-63 x 32-63, 2: queries 32-63 x keys 0-31
__device__ __forceinline__ void add_pairs(const bf16x8 (&vf)[4], uint32_t pb, f32x16& o0, f32x16& o1) {
  o0 = mfma(vf[0], read_k_frag(pb), o0);
  o0 = mfma(vf[1], read_k_frag(pb + 1024), o0);
  o1 = mfma(vf[0], read_k_frag(pb + 4096), o1);
  o1 = mfma(vf[1], read_k_frag(pb + 5120), o1);
  o1 = mfma(vf[2], read_k_frag(pb + 2048), o1);
  o1 = mfma(vf[3], read_k_frag(pb + 3072), o1);
}
// H += K^T (w . V): the chunk's V fragments times the tokens' weights at w (element e of fragment s: token
// 16 s + 8 (e / 4) + 4 half + e % 4); k: the K tile
template <class C>
__device__ __forceinline__ void update_state(f32x16 (&H)[C::DBQ], const bf16x8 (&vf)[4], uint32_t w, uint32_t k, const uint32_t (&kt)[C::DBQ][2]) {
  f32x4 wv[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) wv[s] = lds_read16(w + 32 * s);
  uint32_t ka[C::DBQ][2];
#pragma unroll
  for (int db = 0; db < C::DBQ; ++db)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      ka[db][j] = k + kt[db][j];
      pin(ka[db][j]);
    }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    bf16x8 vw;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      vw[e] = (__bf16)((float)vf[s][e] * wv[2 * s][e]);
      vw[4 + e] = (__bf16)((float)vf[s][4 + e] * wv[2 * s + 1][e]);
    }
#pragma unroll
    for (int db = 0; db < C::DBQ; ++db)
      H[db] = mfma(read_tr_frag(ka[db][0] + 16 * s * C::RBQ, ka[db][1] + 16 * s * C::RBQ), vw, H[db]);
  }
}
// One block of 32 queries x 32 columns, turned around in the wavefront's 4 KB of LDS (16-byte chunk k of row r at k ^ (r % 8)):
// afterwards v[k] holds columns 4 (lane % 8) .. + 3 of row 8 k + lane / 8.
__device__ __forceinline__ void turn_around(uint32_t out, int lane, const f32x16& o, f32x4 (&v)[4]) {
  const int ln = lane & 31, half = lane >> 5, row = lane >> 3;
  uint32_t w = out + ln * 128 + ((half ^ (ln & 7)) << 4), r = out + row * 128 + (((lane & 7) ^ row) << 4);
  pin(w);
  pin(r);
#pragma unroll
  for (int a = 0; a < 4; ++a) lds_write16(w ^ (32 * a), (f32x4){o[4 * a], o[4 * a + 1], o[4 * a + 2], o[4 * a + 3]});
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = lds_read16(r + 1024 * k);
}

// ---- the helpers' shares ----
// The gates' values of a chunk (lane = token): a: log-decay, k: key gate (both 0 past the end), s: the factor on the output row.
// Returns the sum of the chunk's log-decays.
template <class C, bool STATE_ONLY>
__device__ __forceinline__ float put_factors(uint32_t gate, int lane, int odd, float a, float k, float s) {
  // b: inclusive prefix sum over the 64 tokens (data-parallel-primitive steps: within rows of 16 lanes by shifts of
  // 1, 2, 4, 8, then the row totals onward)
  float bcum = a;
  bcum += dpp_f<0x111, 0xf, 0xf>(bcum);
  bcum += dpp_f<0x112, 0xf, 0xf>(bcum);
  bcum += dpp_f<0x114, 0xf, 0xe>(bcum);
  bcum += dpp_f<0x118, 0xf, 0xc>(bcum);
  bcum += dpp_f<0x142, 0xa, 0xf>(bcum);
  bcum += dpp_f<0x143, 0xc, 0xf>(bcum);
  const float b_last = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, bcum), 63));
  lds_store4(gate + (C::kW + odd * 64 + lane) * 4, k * __expf(b_last - bcum));
  lds_store4(gate + (C::kDec + odd) * 4, __expf(b_last));
  if constexpr (!STATE_ONLY) {
    // Weights inside the chunk, factorised per group of four tokens: with ref_j the sum in front of token j's group
    // (ref_j >= b_i for every i in or behind the group),  e^{b_i - b_j} g_j = e^{b_i - ref_j} * u_j,
    // u_j = g_j e^{ref_j - b_j}: one exponential per token here and four per lane and block of weights instead of
    // one per weight.  ref_j - b_j is at most four log-decays: with the bound of 20 above u_j stays finite.
    const float ref = dpp_f<0x00, 0xf, 0xf>(bcum - a);  // the sum in front of lane (lane & ~3): quad broadcast of the exclusive sum
    lds_store4(gate + (C::kB + lane) * 4, bcum);
    lds_store4(gate + (C::kU + lane) * 4, k * __expf(ref - bcum));
    lds_store4(gate + (C::kS + lane) * 4, s);
    lds_store4(gate + (C::kRef + (lane >> 2)) * 4, ref);
  }
  return b_last;
}
// scores of a 32 x 32 block; k, q: the lane's addresses of their first row fragments
template <class C>
__device__ __forceinline__ f32x16 block_scores(uint32_t k, uint32_t q) {
  pin(k);
  pin(q);
  f32x16 s = zero16();
#pragma unroll
  for (int t = 0; t < C::T; ++t) s = mfma(read_k_frag(k ^ (32 * t)), read_k_frag(q ^ (32 * t)), s);
  return s;
}
// weights of the block: scale e^{b_i - b_j} g_j (q_i . k_j) for key j <= query i (positions inside the chunk), else 0; inside a
// diagonal block keys behind the lane's query (last_key) get weight 0
template <class C>
__device__ __forceinline__ void block_weights(const f32x16& sc, float scale, uint32_t gate, int lane, int kb, int qb, int last_key, uint32_t dst) {
  const int ln = lane & 31, half = lane >> 5;
  const float bi = lds_read4(gate + (C::kB + 32 * qb + ln) * 4);
  float ref[4];
  f32x4 uj[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    ref[a] = lds_read4(gate + (C::kRef + 8 * kb + 2 * a + half) * 4);
    uj[a] = lds_read16(gate + (C::kU + 32 * kb + 8 * a + 4 * half) * 4);
  }
  u32x4 pk[2];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    // (groups past the lane's query have bi > ref: whatever the factor becomes there, the mask below discards it)
    const float qfac = scale * __expf(bi - ref[a]);
    float x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[e] = sc[4 * a + e] * (qfac * uj[a][e]);
      if (8 * a + 4 * half + e > last_key) x[e] = 0.f;
    }
    bf16x2 lo, hi;
    lo[0] = (__bf16)x[0];
    lo[1] = (__bf16)x[1];
    hi[0] = (__bf16)x[2];
    hi[1] = (__bf16)x[3];
    pk[a / 2][2 * (a % 2)] = __builtin_bit_cast(uint32_t, lo);
    pk[a / 2][2 * (a % 2) + 1] = __builtin_bit_cast(uint32_t, hi);
  }
  lds_write16(dst + lane * 16, __builtin_bit_cast(f32x4, pk[0]));
  lds_write16(dst + lane * 16 + 1024, __builtin_bit_cast(f32x4, pk[1]));
}

// The copies of one helper: the tile of a chunk (64 rows of 16 CPR bytes) of each of TILES tensors.  A copy instruction moves
// 1 KB; per instruction of a tile the lane's byte offset inside a chunk is fixed (row r of the tile, 16-byte chunk with the
// tile's swizzle) and the chunk's first row moves the wave-uniform base pointer.  The last chunk, if short, takes the rows past
// its end from the last token (their gates are zero).
template <int CPR, int TILES>
struct TileCopy {
  static constexpr int N = CPR * TILES, CH = 64;  // instructions per chunk
  const __bf16* base;
  int64_t tile_step;
  uint32_t lds_off;
  int lane, L;
  bool rev;
  uint32_t off[CPR];
  __device__ __forceinline__ TileCopy(const __bf16* base_, int64_t tile_step_, uint32_t lds_off_, int lane_, int L_, bool rev_)
      : base(base_), tile_step(tile_step_), lds_off(lds_off_), lane(lane_), L(L_), rev(rev_) {
#pragma unroll
    for (int i = 0; i < CPR; ++i) off[i] = lane_off(i, CH);
  }
  __device__ __forceinline__ uint32_t lane_off(int nb, int rows) const {
    const int pos = nb * 64 + lane, r = pos / CPR, pc = pos % CPR;
    // walking backwards, tile row r is the token r in front of the chunk's first one, and the base pointer stands at
    // the chunk's lowest address: its last row (row 63 of a whole chunk, token 0 of a short one)
    int row = min(r, rows - 1);
    if (rev) row = rows - 1 - row;
    return (uint32_t)(row * (CPR * 16) + ((pc ^ bswz<CPR>(r)) << 4));
  }
  // (shift: elements from `base` to the tensor meant)
  __device__ __forceinline__ void issue(int c, uint32_t stage, int64_t shift = 0) const {
    const int t0 = c * CH, rows = min(L - t0, CH);
    const int64_t r0 = rev ? max(L - CH - t0, 0) : t0;  // the chunk's row with the lowest address
    static_for<0, TILES>([&](auto tc) {
      const __bf16* src = base + shift + decltype(tc)::value * tile_step + r0 * (CPR * 8);
      const uint32_t dst = stage + lds_off + decltype(tc)::value * (CPR * 1024);
      if (rows == CH) {
        static_for<0, CPR>([&](auto nb) { dma16_at<decltype(nb)::value * 1024>(src, off[decltype(nb)::value], dst); });
      } else {
        static_for<0, CPR>([&](auto nb) { dma16_at<decltype(nb)::value * 1024>(src, lane_off(decltype(nb)::value, rows), dst); });
      }
    });
  }
};

// STATE_ONLY: no outputs, only the state update is walked (see GatedParams::state_only): no queries, no weights, one barrier
// per chunk.
// block: the workgroup's number among those of this walk; const_decay(h): the log-decay of head h where p.log_decay is null.
// OUT_GATE: output rows have a factor of their own (1 without GatedParams::gate_on_output).  Not a run-time test: that took 117 us
// for 113 at 8 x 16 heads x 4096, 64/64, where there is none.
// PART: see GatedParams::part.
template <class C, bool STATE_ONLY, bool OUT_GATE, bool PART, class F>
__device__ __forceinline__ void gated_walk(const GatedParams& p, int block, uint32_t lds0, F&& const_decay) {
  using Y = GLayout<C, STATE_ONLY>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ln = lane & 31, half = lane >> 5;
  // workgroup -> batch entry and HPW consecutive value heads of one q/k group, and the segment of the walk
  const int seg = block % p.nseg;
  const int bh0 = (block / p.nseg) * C::HPW, b = bh0 / p.H, h0 = bh0 % p.H;
  const int hqk = h0 / (p.H / p.H_qk);
  const bool rev = p.reverse != 0;
  // the tokens this workgroup walks: L of them from position `first` of the walk (the whole sequence unless it is
  // cut into segments); row_lo: the one with the lowest address, where all base pointers below stand
  const int64_t Lt = p.L, first = (PART ? p.seg_from : 0) + (int64_t)seg * p.seg_len;
  const int L = (int)(PART ? min(p.seg_to - first, (int64_t)p.seg_len) : p.nseg > 1 ? min(Lt - first, (int64_t)p.seg_len) : Lt);
  const int in_slots = PART ? p.in_slots : p.nseg, out_slots = PART ? p.out_slots : p.nseg;  // states of a (batch, head)
  const int64_t row_lo = rev ? Lt - first - L : first;
  const int n_chunks = (L + C::CH - 1) / C::CH;
  auto stage_of = [&](int c) { return lds0 + (uint32_t)(c % Y::STAGES) * Y::STAGE_BYTES; };
  auto gates_of = [&](int hh) { return lds0 + Y::kGates + hh * C::GATE_BYTES; };

  if (wave < C::SW) {
    // ================= state wavefront: 32 value columns of one head =================
    const int hw = wave / C::NB, vblk = wave % C::NB, bh = bh0 + hw;
    const uint32_t gate = gates_of(hw);
    f32x16 H[C::DBQ];  // register r of tile db: row d = 32 db + 16 (r / 8) + 8 half + r % 8 of the slab, column ln
    auto h_row = [&](int db, int r) { return (int64_t)(32 * db + 16 * (r >> 3) + 8 * half + (r & 7)) * C::DV; };
#pragma unroll
    for (int db = 0; db < C::DBQ; ++db) {
      if (p.h_in) {
        const float* src = p.h_in + ((int64_t)bh * in_slots + seg) * C::DQK * C::DV + 32 * vblk + ln;
#pragma unroll
        for (int r = 0; r < 16; ++r) H[db][r] = src[h_row(db, r)];
      } else {
        H[db] = zero16();
      }
      pin(H[db]);
    }
    uint32_t kt0[C::DBQ][2], vt0[2];
    const uint32_t rq0 = row_lane<C>(lane);
#pragma unroll
    for (int k = 0; k < C::DBQ; ++k)
#pragma unroll
      for (int j = 0; j < 2; ++j) kt0[k][j] = tr_lane<C::CPRQ>(lane, k, j, swapped_piece(lane));
#pragma unroll
    for (int j = 0; j < 2; ++j) vt0[j] = Y::kV + hw * C::V_BYTES + tr_lane<C::CPRV>(lane, vblk, j, lane & 3);
    auto update = [&](int c, const bf16x8 (&vf)[4]) {
      update_state<C>(H, vf, gate + (C::kW + (c & 1) * 64 + 4 * half) * 4, stage_of(c) + Y::kK, kt0);
    };
    auto v_frags = [&](int c, bf16x8 (&vf)[4]) {
      uint32_t a0 = stage_of(c) + vt0[0], a1 = stage_of(c) + vt0[1];
      pin(a0);
      pin(a1);
#pragma unroll
      for (int s = 0; s < 4; ++s) vf[s] = read_tr_frag(a0 + 16 * s * C::RBV, a1 + 16 * s * C::RBV);
    };

    if constexpr (STATE_ONLY) {
      chunk_barrier();
      for (int c = 0; c < n_chunks; ++c) {
        const float dec = lds_read4(gate + (C::kDec + (c & 1)) * 4);
        bf16x8 vf[4];
        v_frags(c, vf);
#pragma unroll
        for (int db = 0; db < C::DBQ; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) H[db][r] *= dec;
        update(c, vf);
        chunk_barrier();
      }
    } else {
      chunk_barrier();
      chunk_barrier();
      // eight rows at a time: their lowest address is the same for all lanes, the rest of it the lane's own
      const int64_t o_head = (int64_t)bh * Lt + row_lo;
      const int o_log = p.out_bf16 ? 1 : 2;
      const uint32_t o_lane = (uint32_t)((rev ? 7 - (lane >> 3) : lane >> 3) * C::DV + 4 * (lane & 7)) << o_log;
      for (int c = 0; c < n_chunks; ++c) {
        const uint32_t sb = stage_of(c);
        const int t0 = c * C::CH;
        // ---- read-out of the state in front of the chunk: O^T = H^T Q^T, times scale e^{b_i} ----
        const float dec = lds_read4(gate + (C::kDec + (c & 1)) * 4);
        const float f0 = p.scale * __expf(lds_read4(gate + (C::kB + ln) * 4));
        const float f1 = p.scale * __expf(lds_read4(gate + (C::kB + 32 + ln) * 4));
        // (factors of the finished rows, in 32 bits: on the weights they would take part in the rounding to bf16)
        float g0 = 1.f, g1 = 1.f;
        if constexpr (OUT_GATE) {
          g0 = lds_read4(gate + (C::kS + ln) * 4);
          g1 = lds_read4(gate + (C::kS + 32 + ln) * 4);
        }
        f32x16 o0, o1;
        read_out<C>(H, dec, sb + rq0, o0, o1);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          o0[r] *= f0;
          o1[r] *= f1;
        }
        chunk_barrier();
        // ---- the chunk's own tokens ----
        bf16x8 vf[4];
        v_frags(c, vf);
        add_pairs(vf, lds0 + Y::kP + hw * C::P_BYTES + lane * 16, o0, o1);
        if constexpr (OUT_GATE) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            o0[r] *= g0;
            o1[r] *= g1;
          }
        }
        // ---- store ----
        const uint32_t out = Y::kOutInQ ? sb + wave * 4096 : lds0 + Y::kOut + wave * 4096;
        auto store_block = [&](auto ibc, const f32x16& o) {
          constexpr int IB = decltype(ibc)::value;
          f32x4 v[4];
          turn_around(out, lane, o, v);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int i0 = t0 + 32 * IB + 8 * k;
            if (lane >> 3 < L - i0) {
              char* dst = static_cast<char*>(p.O) + (((o_head + (rev ? L - 8 - i0 : i0)) * C::DV + 32 * vblk) << o_log) + o_lane;
              if (p.out_bf16) {
                bf16x4 hv;
#pragma unroll
                for (int e = 0; e < 4; ++e) hv[e] = (__bf16)v[k][e];
                *reinterpret_cast<bf16x4*>(dst) = hv;
              } else {
                *reinterpret_cast<f32x4*>(dst) = v[k];
              }
            }
          }
        };
        store_block(std::integral_constant<int, 0>{}, o0);
        store_block(std::integral_constant<int, 1>{}, o1);
        update(c, vf);
        chunk_barrier();
      }
    }
    if (p.h_out && (!p.h_out_last_only || seg == p.nseg - 1)) {
      float* dst = p.h_out + (p.h_out_last_only ? (int64_t)bh : (int64_t)bh * out_slots + seg) * C::DQK * C::DV + 32 * vblk + ln;
#pragma unroll
      for (int db = 0; db < C::DBQ; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) dst[h_row(db, r)] = H[db][r];
    }
    return;
  }

  const int role = wave - C::SW;
  if (role == 3) {
    // ================= the gates: lane = token of the chunk =================
    float la[C::HPW], g[C::HPW], seg_b[C::HPW];
    auto load_gates = [&](int c) {
      const int t = c * C::CH + lane, gi = min(t, L - 1);
      // walking backwards: the decay of the token one later in the sequence (the walk's first token has none: its
      // value is replaced by 0; cut into segments, the first token of a later segment does have a successor: the
      // word behind the segment), the gate of the token itself
      const int gl = rev ? min(L - gi, first > 0 ? L : L - 1) : gi, gg = rev ? L - 1 - gi : gi;
#pragma unroll
      for (int hh = 0; hh < C::HPW; ++hh) {
        const int64_t row = (int64_t)(bh0 + hh) * Lt + row_lo;
        la[hh] = p.log_decay ? p.log_decay[row + gl] : const_decay(h0 + hh);
        g[hh] = p.key_gate ? p.key_gate[row + gg] : 1.f;
      }
    };
    auto put_gates = [&](int c) {
      const int t = c * C::CH + lane;
#pragma unroll
      for (int hh = 0; hh < C::HPW; ++hh) {
        const uint32_t gate = gates_of(hh);
        // log-decay (0 past the end: the state is carried unchanged; at least -20: a token that lets less than e^-20
        // through lets nothing through at the precision of the path, and the bound keeps the factorised weights below in
        // range) and key gate (0 past the end); a constant decay is the same for every token: nothing to shift or to bound
        float a = la[hh], k = g[hh], s = 1.f;
        if (p.log_decay) a = rev && t == 0 && first == 0 ? 0.f : fmaxf(a, -20.f);
        if (p.gate_on_output) {  // the gate as a factor on the output rows instead of the keys
          s = k;
          k = 1.f;
        }
        if (t >= L) a = k = 0.f;
        seg_b[hh] += put_factors<C, STATE_ONLY>(gate, lane, c & 1, a, k, s);
      }
    };
#pragma unroll
    for (int hh = 0; hh < C::HPW; ++hh) seg_b[hh] = 0.f;
    load_gates(0);
    if constexpr (!STATE_ONLY) chunk_barrier();
    put_gates(0);
    if (n_chunks > 1) load_gates(1);
    chunk_barrier();
    for (int c = 0; c < n_chunks; ++c) {
      if constexpr (!STATE_ONLY) chunk_barrier();
      if (c + 1 < n_chunks) {
        put_gates(c + 1);
        if (c + 2 < n_chunks) load_gates(c + 2);
      }
      chunk_barrier();
    }
    if (p.seg_decay && lane == 0) {
#pragma unroll
      for (int hh = 0; hh < C::HPW; ++hh) p.seg_decay[(int64_t)(bh0 + hh) * out_slots + seg] = seg_b[hh];
    }
    return;
  }

  // ================= copies (helper 0: Q, 1: K, 2: V of every head) and weights =================
  // scores of this helper's block in front of the weights: role 0: keys 0-31 x queries 0-31, 1: 32-63 x 32-63, 2: 0-31 x 32-63
  const int kb = role == 1 ? 1 : 0, qb = role == 0 ? 0 : 1;
  const int last_key = role == 2 ? C::CH : ln;  // inside a diagonal block keys behind the lane's query get weight 0
  const uint32_t rq0 = row_lane<C>(lane);
  auto scores = [&](int c) { return block_scores<C>(stage_of(c) + Y::kK + 32 * kb * C::RBQ + rq0, stage_of(c) + 32 * qb * C::RBQ + rq0); };
  auto weigh = [&](const f32x16& sc) {
#pragma unroll
    for (int hh = 0; hh < C::HPW; ++hh) block_weights<C>(sc, p.scale, gates_of(hh), lane, kb, qb, last_key, lds0 + Y::kP + hh * C::P_BYTES + role * 2048);
  };
  auto help = [&](const auto& cp) {
    constexpr int N = std::decay_t<decltype(cp)>::N;
    if constexpr (STATE_ONLY) {
      // this wavefront's share of chunk c has landed: all of its copies but those of the chunks behind it (at most two)
      auto landed = [&](int c) {
        const int behind = min(n_chunks - 1 - c, 2);
        if (behind == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * N) : "memory");
        else if (behind == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      };
      for (int c = 0; c < min(n_chunks, 3); ++c) cp.issue(c, stage_of(c));
      landed(0);
      chunk_barrier();
      for (int c = 0; c < n_chunks; ++c) {
        if (c + 3 < n_chunks) cp.issue(c + 3, stage_of(c + 3));
        if (c + 1 < n_chunks) landed(c + 1);
        chunk_barrier();
      }
    } else {
      auto landed = [&](bool one_behind) {
        if (one_behind) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      };
      cp.issue(0, stage_of(0));
      if (n_chunks > 1) cp.issue(1, stage_of(1));
      landed(n_chunks > 1);
      chunk_barrier();
      f32x16 s = scores(0);
      chunk_barrier();
      for (int c = 0; c < n_chunks; ++c) {
        const bool more = c + 2 < n_chunks;
        if (more) cp.issue(c + 2, stage_of(c + 2));
        weigh(s);
        if (c + 1 < n_chunks) landed(more);
        chunk_barrier();
        if (c + 1 < n_chunks) s = scores(c + 1);
        chunk_barrier();
      }
    }
  };
  const int64_t qk_row = ((int64_t)b * p.H_qk + hqk) * Lt + row_lo;
  if (role == 2) {
    // (HPW > 1: the heads' V are consecutive, see launch_gated_recurrent)
    const int64_t v_row = ((int64_t)b * p.H_v + h0 / (p.H / p.H_v)) * Lt + row_lo;
    help(TileCopy<C::CPRV, C::HPW>(p.V + v_row * C::DV, Lt * C::DV, Y::kV, lane, L, rev));
  } else if (role == 1 || !STATE_ONLY) {
    help(TileCopy<C::CPRQ, 1>((role == 1 ? p.K : p.Q) + qk_row * C::DQK, 0, role == 1 ? Y::kK : 0, lane, L, rev));
  } else {
    for (int c = 0; c <= n_chunks; ++c) chunk_barrier();
  }
}

template <class C, bool STATE_ONLY>
__global__ __launch_bounds__(C::BOUND_THREADS, C::WAVES_PER_SIMD) void gated_recurrent_kernel(const GatedParams p, const DecayTable dt, int first_block) {
  __shared__ __attribute__((aligned(1024))) char smem[GLayout<C, STATE_ONLY>::LDS_BYTES];
  gated_walk<C, STATE_ONLY, false, false>(p, first_block + (int)blockIdx.x, (uint32_t)(uintptr_t)((lds_char*)smem),
                                   [&](int h) { return dt.log2_gamma[h] * 0.6931471805599453f; });  // ln gamma
}

// See launch_gated_lead.  The longer workgroups come first.
template <class C>
__global__ __launch_bounds__(C::BOUND_THREADS, C::WAVES_PER_SIMD) void gated_lead_kernel(const GatedParams lead, const GatedParams states, const DecayTable dt,
                                                                                          int lead_blocks) {
  constexpr int A = GLayout<C, false>::LDS_BYTES, B = GLayout<C, true>::LDS_BYTES;
  __shared__ __attribute__((aligned(1024))) char smem[A > B ? A : B];
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_char*)smem);
  const int block = (int)blockIdx.x;
  const auto decay = [&](int h) { return dt.log2_gamma[h] * 0.6931471805599453f; };
  if (block < lead_blocks) gated_walk<C, false, false, true>(lead, block, lds0, decay);
  else gated_walk<C, true, false, true>(states, block - lead_blocks, lds0, decay);
}
// Segments of a part of the walk in full.
template <class C>
__global__ __launch_bounds__(C::BOUND_THREADS, C::WAVES_PER_SIMD) void gated_part_kernel(const GatedParams p, const DecayTable dt) {
  __shared__ __attribute__((aligned(1024))) char smem[GLayout<C, false>::LDS_BYTES];
  gated_walk<C, false, false, true>(p, (int)blockIdx.x, (uint32_t)(uintptr_t)((lds_char*)smem), [&](int h) { return dt.log2_gamma[h] * 0.6931471805599453f; });
}

// ---- backward pass where value heads share a q/k head: the gradients of q and k, summed over heads ----
// The walk of gated_recurrent_kernel for several value heads of one q/k head in one workgroup, which takes them in turn, chunk
// by chunk: a unit of work is a (chunk, head).  Queries and keys of the walk (dO and V) are each head's own and arrive per unit,
// the values (K, or Q in the walk that goes backwards) and the rows of the dot products (Q, or K) once per
// chunk.  The outputs are summed over the heads in registers, and each head's row products
// (q . dq, k . dk / g) are formed on the way.  Stored per head, as gated_bwd_rows_kernel takes them, the two walks wrote and that
// kernel read 2 x 251 MB at 8 x 80 heads x 768 tokens: 379 us for the whole backward pass with a launch per walk, 257 this way; with the
// walks in one launch see gated_group_heads.
// DQK_, DV_: head dims of the walk, i.e. of dO and V, and of Q and K.
// HEADS_: at most, per workgroup: 32 registers of state each at head dim 64.  Four need 253 registers, with one address held for each
// kind of fragment and everything else formed from the lane's number in every unit.  Three / four, 128/64: 8 x 80 heads x 768 217 / 196 us
// (27 / 20 parts per gradient), 8 x 64 166 / 142.  Up to three heads have an instance of their own: 8 x 24 x 600 66.0, in that of four 67.7.
template <int DQK_, int DV_, int HEADS_>
struct GroupCfg : GCfg<DQK_, DV_> {
  using G = GCfg<DQK_, DV_>;
  static constexpr int HEADS = HEADS_;
  // what the lane's number gives is hidden from the optimiser, so that it is formed in every unit and not kept through the loop; the
  // rows of the dot products are read one block at a time
  static constexpr bool LEAN = HEADS > 3;
  static constexpr int UNIT_BYTES = 2 * G::Q_BYTES, SHARED_BYTES = 2 * G::V_BYTES;
  static constexpr int kShared = 3 * UNIT_BYTES, kP = kShared + 2 * SHARED_BYTES, kGates = kP + G::P_BYTES;
  static constexpr int kDots = kGates + G::GATE_BYTES, kOut = kDots + G::NB * 256, LDS_BYTES = kOut + G::NB * 4096;
  static_assert(LDS_BYTES <= 160 * 1024, "tiles do not fit LDS");
};

template <class C>
__device__ __forceinline__ void gated_group_walk(const GatedGroupParams& p, int block, uint32_t lds0) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ln = lane & 31, half = lane >> 5;
  const int part = block % p.parts, bhq = block / p.parts, group = p.H / p.H_qk;
  const int nh = min(p.heads, group - part * p.heads);                          // heads of this workgroup
  const int64_t bh0 = (int64_t)bhq * group + part * p.heads;                    // the first of them, batch included
  const bool rev = p.reverse != 0;
  const int L = p.L, n_chunks = (L + C::CH - 1) / C::CH, units = n_chunks * nh;
  const uint32_t gate = lds0 + C::kGates;
  auto unit_stage = [&](int st) { return lds0 + (uint32_t)st * C::UNIT_BYTES; };
  auto shared_stage = [&](int c) { return lds0 + C::kShared + (uint32_t)(c & 1) * C::SHARED_BYTES; };
  auto next = [](int st) { return st == 2 ? 0 : st + 1; };

  if (wave < C::NB) {
    // ================= state wavefront: 32 columns of every head =================
    f32x16 H[C::HEADS][C::DBQ];
#pragma unroll
    for (int n = 0; n < C::HEADS; ++n)
#pragma unroll
      for (int db = 0; db < C::DBQ; ++db) H[n][db] = zero16();
    // (of each kind of fragment one address: block k of 32 columns is at ^ 64 k, the rows 8 further down at (^ 32) + 8 rows)
    uint32_t rq0 = row_lane<C>(lane), kt0 = C::Q_BYTES + tr_lane<C::CPRQ>(lane, 0, 0, swapped_piece(lane)), vt0 = tr_lane<C::CPRV>(lane, wave, 0, lane & 3);
    // the rows of the dot products as the outputs lie in registers: row ln, columns 32 wave + 8 a + 4 half + {0..3} (at ^ 16 a)
    const uint32_t rr0 = C::V_BYTES + ln * C::RBV + (((4 * wave) ^ bswz<C::CPRV>(ln)) << 4) + 8 * half;
    const uint32_t out = lds0 + C::kOut + wave * 4096, dots = lds0 + C::kDots + wave * 256;
    chunk_barrier();
    chunk_barrier();
    int st = 0, odd = 0;  // unit modulo 3 and 2
    for (int c = 0; c < n_chunks; ++c) {
      const uint32_t sh = shared_stage(c);
      const int t0 = c * C::CH;
      f32x16 sum0 = zero16(), sum1 = zero16();
      static_for<0, C::HEADS>([&](auto nc) {
        constexpr int n = decltype(nc)::value;
        if (n < nh) {
          const uint32_t sb = unit_stage(st);
          int lane_now = lane;
          if constexpr (C::LEAN) pin(lane_now);
          const int ln = lane_now & 31, half = lane_now >> 5;
          const float dec = lds_read4(gate + (C::kDec + odd) * 4);
          const float f0 = p.scale * __expf(lds_read4(gate + (C::kB + ln) * 4));
          const float f1 = p.scale * __expf(lds_read4(gate + (C::kB + 32 + ln) * 4));
          const float g0 = lds_read4(gate + (C::kS + ln) * 4), g1 = lds_read4(gate + (C::kS + 32 + ln) * 4);
          f32x16 o0, o1;
          read_out<C>(H[n], dec, sb + rq0, o0, o1);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            o0[r] *= f0;
            o1[r] *= f1;
          }
          chunk_barrier();
          // (read anew for every head, and the fences keep the sums in front of the update: registers)
          bf16x8 vf[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) vf[s] = read_tr_frag(sh + vt0 + 16 * s * C::RBV, sh + (vt0 ^ 32u) + 8 * C::RBV + 16 * s * C::RBV);
          bf16x4 rows[C::LEAN ? 1 : 2][4];
          auto read_rows = [&](int q) {
            uint32_t ra = sh + rr0;
            if constexpr (C::LEAN) pin(ra);
#pragma unroll
            for (int a = 0; a < 4; ++a)
              rows[C::LEAN ? 0 : q][a] = *reinterpret_cast<__attribute__((address_space(3))) const bf16x4*>((lds_char*)(uintptr_t)((ra ^ (16u * a)) + 32 * q * C::RBV));
          };
          read_rows(0);
          if constexpr (!C::LEAN) read_rows(1);
          add_pairs(vf, lds0 + C::kP + lane_now * 16, o0, o1);
          sched_fence();
          float d0 = 0.f, d1 = 0.f;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            d0 = __builtin_fmaf(o0[r], (float)rows[0][r / 4][r % 4], d0);
            sum0[r] = __builtin_fmaf(g0, o0[r], sum0[r]);
          }
          if constexpr (C::LEAN) {
            sched_fence();
            read_rows(1);
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            sum1[r] = __builtin_fmaf(g1, o1[r], sum1[r]);
            d1 = __builtin_fmaf(o1[r], (float)rows[C::LEAN ? 0 : 1][r / 4][r % 4], d1);
          }
          d0 = sum_halves(d0);
          d1 = sum_halves(d1);
          lds_store4(dots + lane_now * 4, half ? d1 : d0);  // of token `lane` of the chunk
          sched_fence();
          if (n == nh - 1) {
            auto store_block = [&](auto qc, const f32x16& o) {
              f32x4 v[4];
              turn_around(out, lane_now, o, v);
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                const int i = t0 + 32 * decltype(qc)::value + 8 * k + (lane_now >> 3);
                if (i < L)
                  *reinterpret_cast<f32x4*>(p.out + (((int64_t)bhq * p.parts + part) * L + (rev ? L - 1 - i : i)) * C::DV + 32 * wave + 4 * (lane_now & 7)) = v[k];
              }
            };
            store_block(std::integral_constant<int, 0>{}, sum0);
            store_block(std::integral_constant<int, 1>{}, sum1);
          }
          sched_fence();
          uint32_t kt[C::DBQ][2];
          if constexpr (C::LEAN) pin(kt0);
#pragma unroll
          for (int k = 0; k < C::DBQ; ++k) {
            kt[k][0] = kt0 ^ (64u * k);
            kt[k][1] = (kt[k][0] ^ 32u) + 8 * C::RBQ;
          }
          update_state<C>(H[n], vf, gate + (C::kW + odd * 64 + 4 * half) * 4, sb, kt);
          chunk_barrier();
          st = next(st);
          odd ^= 1;
        }
      });
    }
    return;
  }

  const int role = wave - C::NB;
  if (role == 3) {
    // ================= the gates: lane = token of the chunk; and the heads' row products =================
    float la = 0.f, g = 1.f;         // of the unit to prepare next
    float g_put = 1.f, g_done = 1.f;  // of the unit prepared last, of the one whose products are due
    auto token = [&](int c) {
      const int i = min(c * C::CH + lane, L - 1);
      return rev ? L - 1 - i : i;
    };
    auto load = [&](int c, int n) {
      const int64_t row = (bh0 + n) * L;
      const int t = token(c);
      // (walking backwards: the decay of the token one later in the sequence; the walk's first token has none)
      la = p.log_decay[row + (rev ? min(t + 1, L - 1) : t)];
      g = p.key_gate ? p.key_gate[row + t] : 1.f;
    };
    auto put = [&](int c, int odd) {
      const int t = c * C::CH + lane;
      float a = rev && t == 0 ? 0.f : fmaxf(la, -20.f), k = rev ? 1.f : g;
      if (t >= L) a = k = 0.f;
      put_factors<C, false>(gate, lane, odd, a, k, rev ? g : 1.f);
    };
    auto finish = [&](int c, int n) {
      float d = 0.f;
#pragma unroll
      for (int w = 0; w < C::NB; ++w) d += lds_read4(lds0 + C::kDots + w * 256 + lane * 4);
      if (c * C::CH + lane < L) {
        const int64_t e = (bh0 + n) * L + token(c);
        if (rev) {
          if (p.dkey_gate) p.dkey_gate[e] = d;
          d *= g_done;
        }
        p.dots[e] = d;
      }
    };
    int c = 0, n = 0, cl = 0, nl = 0, cd = 0, nd = 0;  // the unit under way, the next to load, the next to finish
    auto step = [&](int& cc, int& nn) {
      if (++nn == nh) {
        nn = 0;
        ++cc;
      }
    };
    load(0, 0);
    step(cl, nl);
    chunk_barrier();
    put(0, 0);
    g_put = g;
    if (units > 1) load(cl, nl);
    chunk_barrier();
    for (int u = 0; u < units; ++u) {
      if (u > 0) {
        finish(cd, nd);
        step(cd, nd);
      }
      chunk_barrier();
      g_done = g_put;
      step(c, n);
      if (u + 1 < units) {
        put(c, (u + 1) & 1);
        g_put = g;
        step(cl, nl);
        if (u + 2 < units) load(cl, nl);
      }
      chunk_barrier();
    }
    finish(cd, nd);
    return;
  }

  // ================= copies (helper 0: queries, 1: keys of a unit, 2: values and rows of a chunk) and weights =================
  const int kb = role == 1 ? 1 : 0, qb = role == 0 ? 0 : 1;
  const int last_key = role == 2 ? C::CH : ln;
  const uint32_t rq0 = row_lane<C>(lane);
  auto scores = [&](int st) { return block_scores<C>(unit_stage(st) + C::Q_BYTES + 32 * kb * C::RBQ + rq0, unit_stage(st) + 32 * qb * C::RBQ + rq0); };
  auto help = [&](auto&& start, auto&& copy, auto&& landed) {
    start();
    chunk_barrier();
    int st = 0;
    f32x16 s = scores(0);
    chunk_barrier();
    for (int u = 0; u < units; ++u) {
      copy(u);
      block_weights<C>(s, p.scale, gate, lane, kb, qb, last_key, lds0 + C::kP + role * 2048);
      landed(u);
      chunk_barrier();
      st = next(st);
      if (u + 1 < units) s = scores(st);
      chunk_barrier();
    }
  };
  if (role == 2) {
    const int64_t row = (int64_t)bhq * L * C::DV;
    TileCopy<C::CPRV, 2> cp(p.V + row, (int64_t)((intptr_t)p.R - (intptr_t)p.V) / 2, 0, lane, L, rev);
    int c = 0, n = 0;
    help([&] { cp.issue(0, shared_stage(0)); },
         [&](int) {
           if (n == 0) {  // the chunk's tiles have landed (they are used behind the next barrier), the next chunk's follow
             asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
             if (c + 1 < n_chunks) cp.issue(c + 1, shared_stage(c + 1));
           }
           if (++n == nh) {
             n = 0;
             ++c;
           }
         },
         [](int) {});
  } else {
    const int64_t head = (int64_t)L * C::DQK;
    TileCopy<C::CPRQ, 1> cp((role == 1 ? p.K : p.Q) + bh0 * head, 0, role == 1 ? C::Q_BYTES : 0, lane, L, rev);
    int c = 0, n = 0, st = 0;  // the unit to copy next
    auto issue = [&] {
      cp.issue(c, unit_stage(st), n * head);
      st = next(st);
      if (++n == nh) {
        n = 0;
        ++c;
      }
    };
    auto wait = [&](bool one_behind) {
      if (one_behind) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(C::CPRQ) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    help(
        [&] {
          issue();
          if (units > 1) issue();
          wait(units > 1);
        },
        [&](int u) {
          if (u + 2 < units) issue();
        },
        [&](int u) {
          if (u + 1 < units) wait(u + 2 < units);
        });
  }
}

// ---- the three walks of the backward pass in one launch ----
// They do not depend on each other, each is a chain of chunks as long as the sequence, and with a launch for each the next one
// waits for the last workgroup of the one before.  Side by side they fill the compute units that one of them leaves idle.
// Three launches / one (us): 1 x 8 heads x 768, 128/128, 66.6 / 32.3, 2 x 32 x 768 120 / 57, 4 x 32 x 768 131 / 103,
// 8 x 32 x 768 203 / 195, 4 x 8 x 500 64/64 58 / 28, Mamba2 8 x 80 x 768 256 / 224, 1 x 80 x 300 61 / 31.
// A: head dims of the walks for the gradients of q and k (D_v, D_qk), E: of the one for that of v (D_qk, D_v); GATED: with key
// gates, which are factors of the rows of the latter.  The longest
// workgroups come first: GROUP: those that take several heads; otherwise all are alike and the gradient of v, which no
// later kernel reads, goes first (the others are still in the caches then: 8 x 32 x 768 202 against 192).
struct GatedBackwardWalks {
  GatedParams walk[3];
  GatedGroupParams group[2];
  int first[2];     // number of the first workgroup of walks 1 and 2
  int first_block;  // ... and of the launch
};
template <class A, class E, bool STATE_ONLY, bool GROUP>
struct BackwardCfg {
  static constexpr int THREADS = A::THREADS > E::THREADS ? A::THREADS : E::THREADS;
  static constexpr bool SHARES_CU = A::SHARES_CU && E::SHARES_CU && !GROUP;
  static constexpr int WAVES_PER_SIMD = SHARES_CU ? 4 : 2, BOUND_THREADS = SHARES_CU ? 512 : THREADS;
  static constexpr int first_two() {
    if constexpr (GROUP) return A::LDS_BYTES;
    else return GLayout<A, STATE_ONLY>::LDS_BYTES;
  }
  static constexpr int THIRD = GLayout<E, STATE_ONLY>::LDS_BYTES;
  static constexpr int LDS_BYTES = first_two() > THIRD ? first_two() : THIRD;
};
template <class A, class E, bool STATE_ONLY, bool GROUP, bool GATED>
__global__ __launch_bounds__((BackwardCfg<A, E, STATE_ONLY, GROUP>::BOUND_THREADS), (BackwardCfg<A, E, STATE_ONLY, GROUP>::WAVES_PER_SIMD))
void gated_backward_kernel(const GatedBackwardWalks w) {
  typedef BackwardCfg<A, E, STATE_ONLY, GROUP> C;
  __shared__ __attribute__((aligned(1024))) char smem[C::LDS_BYTES];
  const uint32_t lds0 = (uint32_t)(uintptr_t)((lds_char*)smem);
  const int n = w.first_block + (int)blockIdx.x, which = (n >= w.first[0] ? 1 : 0) + (n >= w.first[1] ? 1 : 0);
  const int block = n - (which == 0 ? 0 : w.first[which - 1]);
  const auto no_const = [](int) { return 0.f; };
  constexpr int kE = GROUP ? 2 : 0;  // place of the walk for the gradient of v
  if constexpr (std::is_same<A, E>::value) {
    gated_walk<E, STATE_ONLY, GATED, false>(w.walk[which], block, lds0, no_const);
  } else {
    // (wavefronts beyond those of the walk end here: a barrier counts those that are left)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (which == kE) {
      if (wave < E::WAVES) gated_walk<E, STATE_ONLY, GATED, false>(w.walk[kE], block, lds0, no_const);
    } else if (wave < A::WAVES) {
      if constexpr (GROUP) gated_group_walk<A>(w.group[which], block, lds0);
      else gated_walk<A, STATE_ONLY, false, false>(w.walk[which], block, lds0, no_const);
    }
  }
}

// dQ and dK (blockIdx.y) of every q/k head: the sum of its parts, in their order
__global__ __launch_bounds__(256) void gated_group_sum_kernel(const float* dq_parts, const float* dk_parts, float* dQ, float* dK, int parts,
                                                              int64_t head_elems, int64_t elems) {
  const int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (e >= elems) return;
  const int64_t head = e / head_elems, in = e % head_elems;
  const float* src = (blockIdx.y ? dk_parts : dq_parts) + head * parts * head_elems + in;
  f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int i = 0; i < parts; ++i) x += *reinterpret_cast<const f32x4*>(src + i * head_elems);
  *reinterpret_cast<f32x4*>((blockIdx.y ? dK : dQ) + e) = x;
}

// More workgroups than a launch holds (see launch_fits) go in several: launch(first workgroup, their number) each.
template <class F>
hipError_t launch_in_parts(int64_t blocks, int threads, F&& launch) {
  const int64_t most = 0xffffffffLL / threads;
  hipError_t e = hipSuccess;
  for (int64_t first = 0; first < blocks && e == hipSuccess; first += most) {
    launch((int)first, dim3((unsigned)(blocks - first < most ? blocks - first : most)));
    e = hipGetLastError();
  }
  return e;
}

// LDS that a launch asks for on top, so that workgroups which could share a compute unit have one each (see gated_one_each).
static int lds_for_one_each(bool one_each) { return one_each ? 1024 : 0; }

template <int DQK, int DV, int HPW = 1>
hipError_t launch(const GatedParams& p, const DecayTable& dt, hipStream_t s) {
  typedef GCfg<DQK, DV, HPW> C;
  if (p.gate_on_output && !p.state_only) return hipErrorInvalidValue;
  const int64_t blocks = (int64_t)p.B * p.H / HPW * p.nseg;
  if (p.part) {
    if (p.state_only || !launch_fits(blocks, C::THREADS)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gated_part_kernel<C>, dim3((unsigned)blocks), dim3(C::THREADS), 0, s, p, dt);
    return hipGetLastError();
  }
  const int lds = lds_for_one_each(C::SHARES_CU && p.nseg == 1 && gated_one_each(blocks, p.L));
  return launch_in_parts(blocks, C::THREADS, [&](int first, dim3 grid) {
    if (p.state_only) hipLaunchKernelGGL((gated_recurrent_kernel<C, true>), grid, dim3(C::THREADS), 0, s, p, dt, first);
    else hipLaunchKernelGGL((gated_recurrent_kernel<C, false>), grid, dim3(C::THREADS), lds, s, p, dt, first);
  });
}

// ---- segments: from the final states of the segments (each from a zero start) to the states in front of them ----
// One thread per state element, or four, walks the segments; what it waits for is memory, so the states and decays of up to kAhead
// segments are requested together instead of one at a time, each behind the store of the one before (whole calls with walks cut
// in 7 and in 32 segments 210 -> 206 and 245 -> 233 us), and no more than there are (1 x 128 heads x 1152 tokens, two segments,
// 75.9 us with eight requests, 73.3 so).  Four elements a thread instead of one, and nothing of the last segment read: whole calls of 128 pairs
// (128/128) x 1300 59.3 -> 54.4 us, x 4096 171 -> 166, of 96 x 1100 47.2 -> 43.6; beyond eight segments one element, more wavefronts (V; 8 pairs x 32768, 32
// segments, 88.2 with one, 88.8 with four).
template <int V>
struct StatePiece {
  float x[V];
  __device__ __forceinline__ void load(const float* p) {
    if constexpr (V == 4) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = v[i];
    } else {
      x[0] = *p;
    }
  }
  __device__ __forceinline__ void store(float* p) const {
    if constexpr (V == 4) *reinterpret_cast<f32x4*>(p) = f32x4{x[0], x[1], x[2], x[3]};
    else *p = x[0];
  }
  __device__ __forceinline__ void chain(float d, const StatePiece& local) {
#pragma unroll
    for (int i = 0; i < V; ++i) x[i] = d * x[i] + local.x[i];
  }
};
constexpr int kAhead = 8, kChainThreads = 64;  // (one wavefront: few pairs of small states, 24 x 4096 elements, are 96 workgroups of 256)
template <int V>
__global__ __launch_bounds__(kChainThreads) void gated_combine_segments_kernel(float* buf, const float* seg_decay, const float* h_in, int nseg,
                                                                                int state_elems) {
  const int64_t bh = blockIdx.y;
  const int e = (blockIdx.x * kChainThreads + threadIdx.x) * V;
  if (e >= state_elems) return;
  StatePiece<V> x = {};
  if (h_in) x.load(h_in + bh * state_elems + e);
  float* slot = buf + bh * nseg * state_elems + e;
  const float* dec = seg_decay + bh * nseg;
  for (int s0 = 0; s0 < nseg; s0 += kAhead) {
    StatePiece<V> local[kAhead];
    float d[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (s0 + u >= nseg - 1) break;  // (nothing follows the last segment)
      local[u].load(slot + (int64_t)(s0 + u) * state_elems);
      d[u] = dec[s0 + u];
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (s0 + u >= nseg) break;
      x.store(slot + (int64_t)(s0 + u) * state_elems);
      if (s0 + u < nseg - 1) x.chain(__expf(d[u]), local[u]);
    }
  }
}
// The same behind a lead, see launch_gated_chain_segments.
__global__ __launch_bounds__(kChainThreads) void gated_chain_segments_kernel(float* buf, const float* seg_decay, int nseg, int state_elems) {
  const int64_t bh = blockIdx.y;
  const int e = (blockIdx.x * kChainThreads + threadIdx.x) * 4;
  if (e >= state_elems) return;
  float* slot = buf + bh * nseg * state_elems + e;
  const float* dec = seg_decay + bh * nseg;
  StatePiece<4> x;
  x.load(slot);
  for (int s0 = 1; s0 < nseg; s0 += kAhead) {
    StatePiece<4> local[kAhead];
    float d[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (s0 + u >= nseg) break;
      local[u].load(slot + (int64_t)(s0 + u) * state_elems);
      d[u] = dec[s0 + u];
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (s0 + u >= nseg) break;
      x.chain(__expf(d[u]), local[u]);
      x.store(slot + (int64_t)(s0 + u) * state_elems);
    }
  }
}

// ---- epilogue of the backward pass ----
// A group of DQK / 4 lanes owns a token (16 bytes of an fp32 row, 8 of a bf16 row, per lane); a wavefront takes
// 64 / (DQK / 4) tokens of one (batch, q/k head) at a time and loops over the value heads of the group.
template <int DQK>
__global__ __launch_bounds__(256) void gated_bwd_rows_kernel(const GatedBwdEpilogueParams p) {
  constexpr int LPR = DQK / 4, TPW = 64 / LPR;
  const int lane = threadIdx.x & 63, sub = lane % LPR;
  const int grp = p.H / p.H_qk;
  const int64_t blocks_per_head = ((int64_t)p.L + 4 * TPW - 1) / (4 * TPW);
  const int64_t bhq = blockIdx.x / blocks_per_head;  // (batch, q/k head)
  const int64_t t = (blockIdx.x % blocks_per_head) * (4 * TPW) + (threadIdx.x >> 6) * TPW + lane / LPR;
  const bool live = t < p.L;
  const int64_t tc = live ? t : p.L - 1;
  const int b = (int)(bhq / p.H_qk), hq = (int)(bhq % p.H_qk);
  const int64_t qrow = (bhq * p.L + tc) * DQK + 4 * sub;
  const bf16x4 q4 = *reinterpret_cast<const bf16x4*>(p.Q + qrow), k4 = *reinterpret_cast<const bf16x4*>(p.K + qrow);
  f32x4 dq = {0.f, 0.f, 0.f, 0.f}, dk = {0.f, 0.f, 0.f, 0.f};
  for (int j = 0; j < grp; ++j) {
    const int64_t bh = (int64_t)b * p.H + (int64_t)hq * grp + j;
    const int64_t row = (bh * p.L + tc) * DQK + 4 * sub;
    const f32x4 u = *reinterpret_cast<const f32x4*>(p.dQu + row), x = *reinterpret_cast<const f32x4*>(p.X + row);
    const float g = p.key_gate ? p.key_gate[bh * p.L + tc] : 1.f;
    float qd = 0.f, kx = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      qd += (float)q4[e] * u[e];
      kx += (float)k4[e] * x[e];
      dq[e] += u[e];
      dk[e] += g * x[e];
    }
#pragma unroll
    for (int s = LPR / 2; s >= 1; s >>= 1) {
      qd += __shfl_xor(qd, s);
      kx += __shfl_xor(kx, s);
    }
    if (live && sub == 0) {
      p.dB[bh * p.L + t] = qd - g * kx;
      if (p.dkey_gate) p.dkey_gate[bh * p.L + t] = kx;
    }
  }
  if (live) {
    // (where dQu is dQ itself the values are already in place; dK is rewritten only if something changed it)
    if (p.dQu != p.dQ) *reinterpret_cast<f32x4*>(p.dQ + qrow) = dq;
    if (p.X != p.dK || p.key_gate) *reinterpret_cast<f32x4*>(p.dK + qrow) = dk;
  }
}

// dlog_decay[t] = sum_{i >= t} dB[i] - minus[i] (minus: null or dlog_decay itself, read in front of the writes): one wavefront per (batch, head) walks from the end in blocks of 256 tokens,
// four per lane; the running total is kept in double (the terms change sign and the sum is long).
__global__ __launch_bounds__(64) void gated_bwd_suffix_sum_kernel(const float* dB, const float* minus, float* dlog_decay, int L) {
  const int lane = threadIdx.x;
  const float* src = dB + (int64_t)blockIdx.x * L;
  const float* sub = minus ? minus + (int64_t)blockIdx.x * L : nullptr;
  float* dst = dlog_decay + (int64_t)blockIdx.x * L;
  double carry = 0.0;
  const int nblk = (L + 255) / 256;
  for (int blk = nblk - 1; blk >= 0; --blk) {
    const int t0 = blk * 256 + 4 * lane;
    float x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = t0 + e < L ? src[t0 + e] - (sub ? sub[t0 + e] : 0.f) : 0.f;
    // suffix sums inside the lane, then over the lanes behind this one
    x[2] += x[3];
    x[1] += x[2];
    x[0] += x[1];
    float tot = x[0];  // inclusive suffix sum over lanes: lane l gets the sum of the totals of lanes >= l
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
      const float o = __shfl_down(tot, s);
      if (lane + s < 64) tot += o;
    }
    const float behind = tot - x[0];  // the lanes strictly behind
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (t0 + e < L) dst[t0 + e] = (float)(carry + (double)(x[e] + behind));
    carry += (double)__shfl(tot, 0);
  }
}

}  // namespace

hipError_t launch_gated_combine_segments(float* buf, const float* seg_decay, const float* h_in, int BH, int nseg, int state_elems,
                                         hipStream_t s) {
  if (BH < 1 || BH > 65535 || nseg < 1 || state_elems < 4 || state_elems % 4 != 0) return hipErrorInvalidValue;
  auto grid = [&](int v) { return dim3((unsigned)((state_elems + v * kChainThreads - 1) / (v * kChainThreads)), (unsigned)BH); };
  if (nseg <= kAhead) hipLaunchKernelGGL(gated_combine_segments_kernel<4>, grid(4), dim3(kChainThreads), 0, s, buf, seg_decay, h_in, nseg, state_elems);
  else hipLaunchKernelGGL(gated_combine_segments_kernel<1>, grid(1), dim3(kChainThreads), 0, s, buf, seg_decay, h_in, nseg, state_elems);
  return hipGetLastError();
}

hipError_t launch_gated_chain_segments(float* buf, const float* seg_decay, int BH, int nseg, int state_elems, hipStream_t s) {
  if (BH < 1 || BH > 65535 || nseg < 2 || state_elems < 4 || state_elems % 4 != 0) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((state_elems + 4 * kChainThreads - 1) / (4 * kChainThreads)), (unsigned)BH);
  hipLaunchKernelGGL(gated_chain_segments_kernel, grid, dim3(kChainThreads), 0, s, buf, seg_decay, nseg, state_elems);
  return hipGetLastError();
}

bool gated_group_supported(int dqk, int dv) { return (dqk == 64 || dqk == 128) && dv == 64; }

hipError_t launch_gated_group_sum(const float* dq_parts, const float* dk_parts, float* dQ, float* dK, int parts, int64_t head_elems,
                                  int64_t elems, hipStream_t s) {
  const int64_t grid = (elems / 4 + 255) / 256;
  if (!launch_fits(grid, 256)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gated_group_sum_kernel, dim3((unsigned)grid, 2), dim3(256), 0, s, dq_parts, dk_parts, dQ, dK, parts, head_elems, elems);
  return hipGetLastError();
}

hipError_t launch_gated_suffix_sum(const float* dB, const float* minus, float* dlog_decay, int BH, int L, hipStream_t s) {
  if (!launch_fits(BH, 64)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gated_bwd_suffix_sum_kernel, dim3((unsigned)BH), dim3(64), 0, s, dB, minus, dlog_decay, L);
  return hipGetLastError();
}

hipError_t launch_gated_backward_epilogue(const GatedBwdEpilogueParams& p, int dqk, hipStream_t s) {
  const int tpb = 4 * (64 / (dqk / 4));
  const int64_t grid = (int64_t)p.B * p.H_qk * (((int64_t)p.L + tpb - 1) / tpb);
  if (!launch_fits(grid, 256) || (dqk != 64 && dqk != 128)) return hipErrorInvalidValue;
  if (dqk == 64) hipLaunchKernelGGL(gated_bwd_rows_kernel<64>, dim3((unsigned)grid), dim3(256), 0, s, p);
  else hipLaunchKernelGGL(gated_bwd_rows_kernel<128>, dim3((unsigned)grid), dim3(256), 0, s, p);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_gated_suffix_sum(p.dB, nullptr, p.dlog_decay, p.B * p.H, p.L, s);
}

bool gated_supported(int dqk, int dv) { return (dqk == 64 || dqk == 128) && (dv == 64 || dv == 128); }

static hipError_t check_walk(GatedParams& p) {
  if (p.H_v == 0) p.H_v = p.H;
  if (p.H_qk < 1 || p.H % p.H_qk != 0 || p.H % p.H_v != 0) return hipErrorInvalidValue;
  const int64_t from = p.part ? p.seg_from : 0, to = p.part ? p.seg_to : p.L;
  if (p.nseg < 1 || from < 0 || from % 64 != 0 || to > p.L ||
      ((p.nseg > 1 || p.part) && (p.seg_len < 64 || p.seg_len % 64 != 0 || from + (int64_t)(p.nseg - 1) * p.seg_len >= to)))
    return hipErrorInvalidValue;
  // value heads that share their q/k head (Mamba2's groups) can share the Q and K tiles of a workgroup, two at a time
  if (p.heads_per_workgroup != 1 && (p.heads_per_workgroup != 2 || p.H / p.H_qk % 2 != 0 || p.H_v != p.H)) return hipErrorInvalidValue;
  return (int64_t)p.B * p.H * p.nseg > 0x7fffffffLL ? hipErrorInvalidValue : hipSuccess;
}

template <int DQK, int DV, int HPW = 1>
static hipError_t launch_lead(const GatedParams& lead, const GatedParams& states, const DecayTable& dt, hipStream_t s) {
  typedef GCfg<DQK, DV, HPW> C;
  const int64_t first = (int64_t)lead.B * lead.H / HPW * lead.nseg, blocks = first + (int64_t)states.B * states.H / HPW * states.nseg;
  if (!launch_fits(blocks, C::THREADS)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gated_lead_kernel<C>, dim3((unsigned)blocks), dim3(C::THREADS), 0, s, lead, states, dt, (int)first);
  return hipGetLastError();
}
hipError_t launch_gated_lead(const GatedParams& lead_in, const GatedParams& states_in, const DecayTable& dt, int dqk, int dv, hipStream_t s) {
  GatedParams lead = lead_in, states = states_in;
  hipError_t e = check_walk(lead);
  if (e == hipSuccess) e = check_walk(states);
  if (e != hipSuccess) return e;
  const bool pairs = lead.heads_per_workgroup == 2;
  if ((pairs && dv != 64) || states.heads_per_workgroup != lead.heads_per_workgroup || !lead.part || !states.part || lead.state_only || !states.state_only || lead.gate_on_output ||
      states.gate_on_output)
    return hipErrorInvalidValue;
  if (dqk == 64 && dv == 64) return pairs ? launch_lead<64, 64, 2>(lead, states, dt, s) : launch_lead<64, 64>(lead, states, dt, s);
  if (dqk == 128 && dv == 64) return pairs ? launch_lead<128, 64, 2>(lead, states, dt, s) : launch_lead<128, 64>(lead, states, dt, s);
  if (dqk == 64 && dv == 128) return launch_lead<64, 128>(lead, states, dt, s);
  if (dqk == 128 && dv == 128) return launch_lead<128, 128>(lead, states, dt, s);
  return hipErrorInvalidValue;
}

hipError_t launch_gated_recurrent(const GatedParams& p_in, const DecayTable& dt, int dqk, int dv, hipStream_t s) {
  GatedParams p = p_in;
  const hipError_t e = check_walk(p);
  if (e != hipSuccess) return e;
  const bool pairs = p.heads_per_workgroup == 2;
  if (pairs && dv != 64) return hipErrorInvalidValue;
  if (dqk == 64 && dv == 64) return pairs ? launch<64, 64, 2>(p, dt, s) : launch<64, 64>(p, dt, s);
  if (dqk == 128 && dv == 64) return pairs ? launch<128, 64, 2>(p, dt, s) : launch<128, 64>(p, dt, s);
  if (dqk == 64 && dv == 128) return launch<64, 128>(p, dt, s);
  if (dqk == 128 && dv == 128) return launch<128, 128>(p, dt, s);
  return hipErrorInvalidValue;
}

template <class A, class E, bool GROUP = false>
static hipError_t launch_walks(GatedBackwardWalks& w, int64_t blocks, hipStream_t s) {
  constexpr int kThreads = BackwardCfg<A, E, false, GROUP>::THREADS;
  static_assert(GROUP || BackwardCfg<A, E, true, false>::THREADS == kThreads, "");
  const bool gated = w.walk[GROUP ? 2 : 0].gate_on_output != 0;
  const int lds = lds_for_one_each(BackwardCfg<A, E, false, GROUP>::SHARES_CU && w.walk[0].nseg == 1 && gated_backward_one_each(blocks, w.walk[0].L));
  return launch_in_parts(blocks, kThreads, [&](int first, dim3 grid) {
    w.first_block = first;
    if constexpr (!GROUP) {
      if (w.walk[0].state_only) {
        hipLaunchKernelGGL((gated_backward_kernel<A, E, true, false, false>), grid, dim3(kThreads), 0, s, w);
        return;
      }
    }
    if (gated) hipLaunchKernelGGL((gated_backward_kernel<A, E, false, GROUP, true>), grid, dim3(kThreads), lds, s, w);
    else hipLaunchKernelGGL((gated_backward_kernel<A, E, false, GROUP, false>), grid, dim3(kThreads), lds, s, w);
  });
}

hipError_t launch_gated_backward(const GatedParams (&walk)[3], const GatedGroupParams* group, int dqk, int dv, hipStream_t s) {
  GatedBackwardWalks w = {};
  const bool pairs = walk[2].heads_per_workgroup == 2;
  if ((pairs && (dv != 64 || walk[0].nseg != 1)) || walk[0].heads_per_workgroup != 1 || walk[1].heads_per_workgroup != 1) return hipErrorInvalidValue;
  int64_t blocks = 0;
  for (int i = 0; i < 3; ++i) {
    const int from = group ? i : (i + 2) % 3;
    GatedParams& p = w.walk[i] = walk[from];
    const hipError_t e = check_walk(p);
    if (e != hipSuccess) return e;
    if (p.nseg != walk[0].nseg || p.state_only != walk[0].state_only) return hipErrorInvalidValue;
    if (i > 0) w.first[i - 1] = (int)blocks;
    if (group && i < 2) {
      const GatedGroupParams& g = w.group[i] = group[i];
      if (!gated_group_supported(dqk, dv) || p.nseg != 1 || p.state_only || g.heads < 1 || g.heads > kGatedGroupHeads || g.H_qk < 1 ||
          g.H % g.H_qk != 0 || (int64_t)g.parts * g.heads < g.H / g.H_qk || (int64_t)(g.parts - 1) * g.heads >= g.H / g.H_qk)
        return hipErrorInvalidValue;
      blocks += (int64_t)g.B * g.H_qk * g.parts;
    } else {
      blocks += (int64_t)p.B * p.H * p.nseg / p.heads_per_workgroup;
    }
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  }
  if (group) {
    auto launch_groups = [&](auto headsc) {
      constexpr int N = decltype(headsc)::value;
      if (dqk == 64) return pairs ? launch_walks<GroupCfg<64, 64, N>, GCfg<64, 64, 2>, true>(w, blocks, s) : launch_walks<GroupCfg<64, 64, N>, GCfg<64, 64>, true>(w, blocks, s);
      return pairs ? launch_walks<GroupCfg<64, 128, N>, GCfg<128, 64, 2>, true>(w, blocks, s) : launch_walks<GroupCfg<64, 128, N>, GCfg<128, 64>, true>(w, blocks, s);
    };
    if (w.group[0].heads == kGatedGroupHeads) return launch_groups(std::integral_constant<int, kGatedGroupHeads>{});
    return launch_groups(std::integral_constant<int, kGatedGroupHeads - 1>{});
  }
  if (pairs) return hipErrorInvalidValue;
  if (dqk == 64 && dv == 64) return launch_walks<GCfg<64, 64>, GCfg<64, 64>>(w, blocks, s);
  if (dqk == 128 && dv == 128) return launch_walks<GCfg<128, 128>, GCfg<128, 128>>(w, blocks, s);
  if (dqk == 64 && dv == 128) return launch_walks<GCfg<128, 64>, GCfg<64, 128>>(w, blocks, s);
  if (dqk == 128 && dv == 64) return launch_walks<GCfg<64, 128>, GCfg<128, 64>>(w, blocks, s);
  return hipErrorInvalidValue;
}

}  // namespace ae
