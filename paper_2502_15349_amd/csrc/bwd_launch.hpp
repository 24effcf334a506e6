// Launch templates of the backward kernels, shared by the per-head-dim instantiation files
// (attn_bwd_<D_qk>_<D_v>.hip), each of which defines one launch_backward_<D_qk>_<D_v>().
#pragma once
#include "bwd.hpp"

namespace ae {
namespace {

// One wavefront per 32 own rows where two workgroups of it fit a CU (64/64, and the query side of 128/128 without a bias
// tensor), a pair of wavefronts elsewhere (the measurements stand at attn_bwd_pair_kernel).  64/64 with a bias tensor has
// both: the pair pays on long walks while an XCD holds no more than one workgroup per CU.  Whole backward pass, one wavefront /
// pair, us: 1 x 6 heads x 1023 x 1060 (8 and 9 workgroups per XCD) 73 / 68, 2 x 12 x 1023 x 1060 (24 and 27) 83 / 80;
// 1 x 6 x 4096 x 4133 (32 and 33) 342 / 398, 8 x 16 x 512 x 549 (64 and 80) 96 / 113, 8 x 16 x 2048 causal (256) 744 / 919,
// without the bias's gradient 364 / 514; 4 x 24 x 100 causal 20.0 / 22.4, 2 x 12 x 512 causal 39.3 / 40.5, unmasked 38.9 / 38.1.
// Causal workgroups are half as long on the average: up to 48 of them (2 x 12 x 2048, 48 and 48, 116 / 109; 4096, 96, 262 / 368).
constexpr int64_t units_per_xcd(bool causal) { return causal ? 48 : 32; }
constexpr int64_t kLongBiasWalk = 384;
// Where only one workgroup fits a CU, short walks stay with one wavefront too: the pair is a tile behind itself, has three tiles
// to wait for at its start, and of a narrow window most waves skip most tiles.  Keys (queries) that a row may see, times the
// q heads that a key-side workgroup walks one after the other.  4 x 24 heads x 4096, one wavefront / pair, us: 128/128 window
// 64 429 / 461, 256 533 / 548, 512 671 / 672; 192/128 64 529 / 572, 256 677 / 686, 512 844 / 827; 128/256 64 635 / 665, 128
// 698 / 705, 256 807 / 778.  Causal without a window: 128/128 64 rows 18.0 / 18.9, 128 28.3 / 28.7, 150 31.3 / 30.4; 192/128
// 21.0 / 21.8, 33.0 / 33.7, 36.4 / 35.8; 128/256 64 rows 23.7 / 24.6, 100 35.0 / 33.8; 128/128 with a bias tensor 64 rows 19.1 / 20.6,
// 100 28.2 / 29.3 (192/128 with one 21.9 / 22.3, 32.8 / 32.3: always pairs).
constexpr int64_t short_window(int dv) { return dv == 256 ? 96 : 256; }
constexpr int64_t short_walk(int dv) { return dv == 256 ? 64 : 128; }

template <int DQK, int DV, int NORM, bool CAUSAL, int OUT, bool BIAS>
hipError_t launch_one(const BwdParams& p, const DecayTable& dt, hipStream_t s) {
  constexpr bool kKvSide = OUT == BWD_DKV;
  constexpr int kOwn = 128;  // (both kernels own 128 rows per workgroup)
  // whole sets of `together` groups per XCD (the kernel's mapping): sets x together x 8 XCDs x workgroups per group
  const int L = kKvSide ? p.L_k : p.L_q;
  const int64_t per_group = (int64_t)((L + kOwn - 1) / kOwn) * (kKvSide ? 1 : p.g);
  const int64_t rounds = ((int64_t)p.B * p.H_kv + 7) / 8, tg = p.together[kKvSide ? 1 : 0];
  const int64_t grid = ((rounds + tg - 1) / tg) * tg * 8 * per_group;
  if (tg < 1 || grid > 0x7fffffffLL) return hipErrorInvalidValue;
  constexpr bool kTwoPerCu = DQK == 64 || (DQK == 128 && DV == 128 && !kKvSide && !BIAS);
  constexpr bool kShort = !kTwoPerCu && CAUSAL && (!BIAS || DQK == 128);
  const int64_t walk = (kKvSide ? (int64_t)p.L_q * p.g : p.L_k), window = p.window < (kKvSide ? p.L_q : p.L_k) ? p.window : 0;
  bool pair = !kTwoPerCu;
  if constexpr (kTwoPerCu && BIAS) pair = rounds * per_group <= units_per_xcd(CAUSAL) && walk / (CAUSAL ? 2 : 1) >= kLongBiasWalk;
  if constexpr (kShort) pair = window ? window * (kKvSide ? p.g : 1) > short_window(DV) : walk > short_walk(DV);
  if constexpr (kTwoPerCu || kShort) {
    typedef BwdCfg<DQK, DV, NORM, CAUSAL, OUT, BIAS> C;
    static_assert(C::OWN == kOwn, "");
    if (!pair) hipLaunchKernelGGL(attn_bwd_kernel<C>, dim3((unsigned)grid), dim3(C::THREADS), 0, s, p, dt);
  }
  if constexpr (!kTwoPerCu || BIAS) {
    typedef BwdPairCfg<DQK, DV, NORM, CAUSAL, OUT, BIAS> C;
    static_assert(C::OWN == kOwn, "");
    if (pair) hipLaunchKernelGGL(attn_bwd_pair_kernel<C>, dim3((unsigned)grid), dim3(C::THREADS), 0, s, p, dt);
  }
  return hipGetLastError();
}

template <int DQK, int DV, int NORM, bool CAUSAL>
hipError_t launch_pair(const BwdParams& p, const DecayTable& dt, hipStream_t s) {
  // the bias tensor comes with softmax, sigmoid and no normalization, and not with head dims 128/256
  constexpr bool kBiasBuilt = (NORM == NORM_SOFTMAX || NORM == NORM_SIGMOID || NORM == NORM_NONE) && !(DQK == 128 && DV == 256);
  if (p.bias != nullptr) {
    if constexpr (kBiasBuilt) {
      const hipError_t e = launch_one<DQK, DV, NORM, CAUSAL, BWD_DKV, true>(p, dt, s);
      if (e != hipSuccess) return e;
      return launch_one<DQK, DV, NORM, CAUSAL, BWD_DQ, true>(p, dt, s);
    } else {
      return hipErrorInvalidValue;
    }
  }
  const hipError_t e = launch_one<DQK, DV, NORM, CAUSAL, BWD_DKV, false>(p, dt, s);
  if (e != hipSuccess) return e;
  return launch_one<DQK, DV, NORM, CAUSAL, BWD_DQ, false>(p, dt, s);
}

template <int DQK, int DV, int NORM>
hipError_t launch_norm(const BwdParams& p, const DecayTable& dt, int causal, hipStream_t s) {
  return causal ? launch_pair<DQK, DV, NORM, true>(p, dt, s) : launch_pair<DQK, DV, NORM, false>(p, dt, s);
}

template <int DQK, int DV>
hipError_t launch_dims(const BwdParams& p, const DecayTable& dt, int norm, int causal, hipStream_t s) {
  switch (norm) {
    case NORM_SOFTMAX: return launch_norm<DQK, DV, NORM_SOFTMAX>(p, dt, causal, s);
    case NORM_SIGMOID: return launch_norm<DQK, DV, NORM_SIGMOID>(p, dt, causal, s);
    case NORM_ABSSUM: return launch_norm<DQK, DV, NORM_ABSSUM>(p, dt, causal, s);
    case NORM_ABS_OF_SUM: return launch_norm<DQK, DV, NORM_ABS_OF_SUM>(p, dt, causal, s);
    case NORM_NONE: return launch_norm<DQK, DV, NORM_NONE>(p, dt, causal, s);
    case BWD_NORM_NONE_RELU: return launch_norm<DQK, DV, BWD_NORM_NONE_RELU>(p, dt, causal, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace
}  // namespace ae
