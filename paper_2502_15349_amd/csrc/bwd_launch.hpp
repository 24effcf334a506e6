// Launch templates of the backward kernels, shared by the per-head-dim instantiation files
// (attn_bwd_<D_qk>_<D_v>.hip), each of which defines one launch_backward_<D_qk>_<D_v>().
#pragma once
#include "bwd.hpp"

namespace ae {
namespace {

// One wavefront per 32 own rows where two workgroups of it share a CU (without a bias tensor: 64/64, and the query side
// of 128/128), a pair of wavefronts elsewhere (the measurements stand at attn_bwd_pair_kernel).
template <int DQK, int DV, int NORM, bool CAUSAL, int OUT, bool BIAS>
struct Choice {
  static constexpr bool PAIR = BIAS || !(DQK == 64 || (DQK == 128 && DV == 128 && OUT == BWD_DQ));
  typedef BwdPairCfg<DQK, DV, NORM, CAUSAL, OUT, BIAS> C;
  static void launch(unsigned grid, const BwdParams& p, const DecayTable& dt, hipStream_t s) {
    if constexpr (PAIR) hipLaunchKernelGGL(attn_bwd_pair_kernel<C>, dim3(grid), dim3(C::THREADS), 0, s, p, dt);
    else hipLaunchKernelGGL((attn_bwd_kernel<BwdCfg<DQK, DV, NORM, CAUSAL, OUT>>), dim3(grid), dim3(256), 0, s, p, dt);
  }
};

template <int DQK, int DV, int NORM, bool CAUSAL, int OUT, bool BIAS>
hipError_t launch_one(const BwdParams& p, const DecayTable& dt, hipStream_t s) {
  typedef Choice<DQK, DV, NORM, CAUSAL, OUT, BIAS> K;
  typedef typename K::C C;  // (both kernels own 128 rows per workgroup)
  // whole sets of `together` groups per XCD (the kernel's mapping): sets x together x 8 XCDs x workgroups per group
  const int L = C::KV_SIDE ? p.L_k : p.L_q;
  const int64_t per_group = (int64_t)((L + C::OWN - 1) / C::OWN) * (C::KV_SIDE ? 1 : p.g);
  const int64_t rounds = ((int64_t)p.B * p.H_kv + 7) / 8, tg = p.together[C::KV_SIDE ? 1 : 0];
  const int64_t grid = ((rounds + tg - 1) / tg) * tg * 8 * per_group;
  if (tg < 1 || grid > 0x7fffffffLL) return hipErrorInvalidValue;
  K::launch((unsigned)grid, p, dt, s);
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
