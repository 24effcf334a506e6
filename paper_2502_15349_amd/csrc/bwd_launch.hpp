// Launch templates of the backward kernels, shared by the per-head-dim instantiation files
// (attn_bwd_<D_qk>_<D_v>.hip), each of which defines one launch_backward_<D_qk>_<D_v>().
#pragma once
#include <algorithm>

#include "bwd.hpp"

namespace ae {
namespace {

// One wavefront per 32 own rows where two workgroups of it fit a CU (64/64, and the query side of 128/128 without a bias
// tensor), a pair of wavefronts elsewhere (the measurements stand at bwd_pair_walk).  64/64 with a bias tensor has
// both: the pair pays on long walks while an XCD holds no more than one workgroup per CU.  Whole backward pass with the bias's gradient, one
// wavefront / pair, us (workgroups per XCD): unmasked 1 x 6 heads x 1023 (16) 40.4 / 34.8, x 2048 (32) 69 / 59, x 3000 (48) 120 / 144, 1 x 16 x 1300 (44) 60 /
// 71, 2 x 12 x 1023 (48) 52 / 62, 8 x 16 x 600 (160) 95 / 115.  Causal workgroups are half as long on the average: 2 x 12 x 768 (36) 41.1 / 38.2, 1 x 6 x 3000 (48)
// 110 / 102, 1 x 16 x 1600 (52) 75.5 / 65.4, x 2048 (64) 108 / 96, 1 x 6 x 4096 (64) 169 / 150, 2 x 12 x 1300 (66) 72.9 / 70.5, x 1600 (78) 86.8 / 95.5, 1 x 16 x 3000
// (96) 229 / 234, 8 x 16 x 768 (192) 114 / 133.
constexpr int64_t units_per_xcd(bool causal) { return causal ? 64 : 32; }
constexpr int64_t kLongBiasWalk = 384;
// Where only one workgroup fits a CU, short causal walks stay with one wavefront too: the pair is a tile behind itself and has three
// tiles to wait for at its start.  Keys (queries) that a row may see, times the q heads that a key-side workgroup walks one after the
// other; the pair's lead over one wavefront is smaller in the abs-sum family and without normalization, and at 128/128 with a bias
// tensor.  8 x 64 heads, one wavefront / pair, us: 192/128 48 rows 40.2 / 41.9, 64 45.7 / 46.4, 80 58.9 / 55.9, 128 75.8 / 73.2, abs-sum 64
// 50.1 / 51.9, 128 80.7 / 83.8, bias tensor 48 46.0 / 47.7, 64 51.3 / 52.0, 100 76.5 / 72.1; 128/256 64 51.4 / 51.3, 80 69.0 / 63.0, abs-sum 64 55.5 / 57.0,
// 128 100.2 / 103.8; 128/128 64 36.3 / 37.7, 80 46.3 / 44.7, 128 60.4 / 59.4, abs-sum 64 40.1 / 41.3, 128 64.4 / 65.0, bias tensor 100 65.3 / 67.8,
// 128 70.0 / 73.6.
template <int DQK, int NORM, bool BIAS>
constexpr int64_t short_walk() { return NORM == NORM_ABSSUM || NORM == NORM_ABS_OF_SUM || NORM == NORM_NONE || (BIAS && DQK == 128) ? 128 : 64; }
// Narrow windows, of which most waves of a pair skip most tiles, count as short at 128/128 only.  4 x 24 heads x 4096, one wavefront / pair:
// 192/128 window 32 498 / 454, 64 488 / 479, 128 541 / 514, 256 624 / 569; 128/256 64 601 / 563, 128 665 / 604; 128/128 64 419 / 427, 128 447 / 450,
// 200 518 / 492, 256 503 / 493.
template <int DQK, int DV>
constexpr int64_t short_window() { return DQK == 128 && DV == 128 ? 128 : 0; }
// Both sides go in one launch (the key side's workgroups first): two launches / one, us, causal unless said: 64/64 1 x 16 heads x
// 1024 54 / 34, 1 x 16 x 4096 186 / 140, 4 x 32/8 x 2048 335 / 289, 8 x 16 x 2048 unmasked 506 / 510, with a bias tensor 2 x 12 x 1023 x 1201
// 85 / 68; 192/128 1 x 16 x 500 53 / 33, 1 x 6 x 4096 259 / 172, 1 x 128 x 4096 2597 / 2607; 128/256 2 x 16 x 1024 100 / 74, 4 x 16 x
// 2048 438 / 433.  Three exceptions:
//   * 64/64 without a bias tensor: alone, the query side has 134 registers, three workgroups per CU; beside the key side it has that
//     one's 202, two.  What the shared launch saves is at its ends: calls of much work (the keys that the query workgroups of an XCD
//     walk, see walked_keys), whose key side fills the device, go one behind the other.  Causal (thousands of walked keys): 1 x 16 x 8192 (524)
//     510 / 490, 1 x 64 x 4096 (524) 535 / 532, 8 x 12 x 4096 (786) 806 / 810, 1 x 32 x 8192 (1049) 970 / 989, 1 x 64 x 8192 (2097) 1963 / 2000; with
//     64 workgroups of the key side per XCD 1 x 128/16 x 4096 (1049) 1207 / 1047, with 128 4 x 32/8 x 4096 1024 / 1027.  Unmasked 8 x 16 x 1024
//     (131) 151 / 146, 1 x 16 x 4096 (262) 249 / 245, 1 x 32 x 4096 (524) 480 / 483, 8 x 64 x 1024 (524) 584 / 593, 8 x 16 x 4096 (2097) 1882 / 1930.
//   * 128/128 without a bias tensor: beside the key side's workgroups those of the query side get a CU each, which they otherwise
//     share by two.  It pays while the key side leaves compute units idle: few workgroups (of 32 compute units per XCD), or
//     causal ones of unequal length.  Causal (workgroups of the key side per XCD): 1 x 16 x 1024 (16) 72 / 43, 1 x 32/8 x 4096 (32) 627 / 529,
//     2 x 12 x 2048 (48) 135 / 124, but 8 x 24/6 x 1000 (48) 287 / 323, 8 x 12 x 700 (72) 102 / 108, 4 x 32/8 x 2048 (64) 519 / 576; unmasked
//     1 x 32/8 x 2048 (16) 305 / 251, 2 x 32/8 x 1500 (24) 282 / 288, 1 x 16 x 2048 (32, 64 of both sides) 136 / 134, but 2 x 32/8 x 2048 (32)
//     441 / 495, 2 x 12 x 2048 (48) 213 / 242.
//   * 192/128, causal, much work: the two sides among each other cost more in the L2 than the ends save (thousands of walked keys; on some
//     cards the long calls are alike either way): 1 x 128 heads x 2048 (262) 766 / 746, 1 x 64 x 4096 (524) 1262 / 1256, 8 x 16 x 2048 (262)
//     760 / 737, 1 x 24 x 8192 (786) 1683 / 1717.
// The workgroups of a side: whole sets of `together` groups (or parts of groups) per XCD (the kernels' mapping): sets x together x
// 8 XCDs x workgroups per group or part.
inline int64_t side_rounds(const BwdParams& p) { return (((int64_t)p.B * p.H_kv << p.cut) + 7) / 8; }
inline int64_t side_per_group(const BwdParams& p, bool key_side) {
  const int64_t n = (int64_t)(((key_side ? p.L_k : p.L_q) + 127) / 128) * (key_side ? 1 : p.g);  // (all kernels own 128 rows per workgroup)
  return (n + (1 << p.cut) - 1) >> p.cut;
}
inline int64_t side_blocks(const BwdParams& p, bool key_side) {
  const int64_t tg = p.together[key_side ? 1 : 0];
  return tg < 1 ? -1 : (side_rounds(p) + tg - 1) / tg * tg * 8 * side_per_group(p, key_side);
}

// The keys that the query side's workgroups of an XCD walk together.
template <bool CAUSAL>
int64_t walked_keys(const BwdParams& p) {
  const int64_t keys = CAUSAL ? p.L_k / 2 : p.L_k;
  return side_rounds(p) * side_per_group(p, false) * std::min<int64_t>(keys, p.window);
}

template <class C>
hipError_t launch_side(const BwdParams& p, const DecayTable& dt, hipStream_t s) {
  const int64_t grid = side_blocks(p, C::KV_SIDE);
  if (!launch_fits(grid, C::THREADS)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(attn_bwd_kernel<C>, dim3((unsigned)grid), dim3(C::THREADS), 0, s, p, dt);
  return hipGetLastError();
}
template <class K, class Q>
hipError_t launch_both(const BwdParams& p, const DecayTable& dt, hipStream_t s) {
  static_assert(K::KV_SIDE && !Q::KV_SIDE && K::OWN == 128 && Q::OWN == 128, "");
  const int64_t key = side_blocks(p, true), query = side_blocks(p, false);
  if (!launch_fits(key, BwdBoth<K, Q>::THREADS) || !launch_fits(query, BwdBoth<K, Q>::THREADS)) return hipErrorInvalidValue;
  auto launch = [&](int64_t blocks, int64_t key_blocks) {
    hipLaunchKernelGGL((attn_bwd_both_kernel<K, Q>), dim3((unsigned)blocks), dim3(BwdBoth<K, Q>::THREADS), 0, s, p, dt, (int)key_blocks);
  };
  if (launch_fits(key + query, BwdBoth<K, Q>::THREADS)) {
    launch(key + query, key);
  } else {
    launch(key, key);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    launch(query, 0);
  }
  return hipGetLastError();
}

template <class K, class Q>
hipError_t launch_sides(const BwdParams& p, const DecayTable& dt, hipStream_t s, bool both) {
  if (both) return launch_both<K, Q>(p, dt, s);
  const hipError_t e = launch_side<K>(p, dt, s);
  return e != hipSuccess ? e : launch_side<Q>(p, dt, s);
}

template <int DQK, int DV, int NORM, bool CAUSAL, bool BIAS>
hipError_t launch_kernels(const BwdParams& p, const DecayTable& dt, hipStream_t s) {
  typedef BwdCfg<DQK, DV, NORM, CAUSAL, BWD_DKV, BIAS> K1;
  typedef BwdCfg<DQK, DV, NORM, CAUSAL, BWD_DQ, BIAS> Q1;
  typedef BwdPairCfg<DQK, DV, NORM, CAUSAL, BWD_DKV, BIAS> K2;
  typedef BwdPairCfg<DQK, DV, NORM, CAUSAL, BWD_DQ, BIAS> Q2;
  const int64_t key_wgs = side_rounds(p) * side_per_group(p, true), workgroups = key_wgs + side_rounds(p) * side_per_group(p, false);  // per XCD
  if constexpr (DQK == 64) {
    if constexpr (BIAS) {
      const int64_t walk = std::min((int64_t)p.L_q * p.g, (int64_t)p.L_k);
      if (workgroups <= units_per_xcd(CAUSAL) && walk / (CAUSAL ? 2 : 1) >= kLongBiasWalk) return launch_both<K2, Q2>(p, dt, s);
    }
    if constexpr (BIAS) return launch_both<K1, Q1>(p, dt, s);
    else return launch_sides<K1, Q1>(p, dt, s, walked_keys<CAUSAL>(p) < (CAUSAL ? 750000 : 500000) || key_wgs < (CAUSAL ? 128 : 64));
  } else {
    auto is_short = [&](int64_t rows, int64_t heads) {
      const int64_t window = p.window < rows ? p.window : 0;
      return window ? window * heads <= short_window<DQK, DV>() : rows * heads <= short_walk<DQK, NORM, BIAS>();
    };
    if constexpr (DQK == 128 && DV == 128 && !BIAS) {
      const bool short_key = CAUSAL && is_short(p.L_q, p.g);
      const bool both = CAUSAL ? key_wgs <= (p.g == 1 ? 48 : 32) : key_wgs <= 24 || workgroups <= 64;
      if constexpr (CAUSAL)
        if (short_key) return launch_sides<K1, Q1>(p, dt, s, both);
      return launch_sides<K2, Q1>(p, dt, s, both);
    } else {
      if constexpr (CAUSAL)
        if (is_short(p.L_q, p.g) && is_short(p.L_k, 1)) return launch_both<K1, Q1>(p, dt, s);
      if constexpr (DQK == 192 && CAUSAL) return launch_sides<K2, Q2>(p, dt, s, walked_keys<true>(p) < 700000 || key_wgs < 64);
      else return launch_both<K2, Q2>(p, dt, s);
    }
  }
}

template <int DQK, int DV, int NORM, bool CAUSAL>
hipError_t launch_bias(const BwdParams& p, const DecayTable& dt, hipStream_t s) {
  // the bias tensor comes with softmax, sigmoid and no normalization, and not with head dims 128/256
  constexpr bool kBiasBuilt = (NORM == NORM_SOFTMAX || NORM == NORM_SIGMOID || NORM == NORM_NONE) && !(DQK == 128 && DV == 256);
  if (p.bias != nullptr) {
    if constexpr (kBiasBuilt) return launch_kernels<DQK, DV, NORM, CAUSAL, true>(p, dt, s);
    else return hipErrorInvalidValue;
  }
  return launch_kernels<DQK, DV, NORM, CAUSAL, false>(p, dt, s);
}

template <int DQK, int DV, bool CAUSAL>
hipError_t launch_mask(const BwdParams& p, const DecayTable& dt, int norm, hipStream_t s) {
  switch (norm) {
    case NORM_SOFTMAX: return launch_bias<DQK, DV, NORM_SOFTMAX, CAUSAL>(p, dt, s);
    case NORM_SIGMOID: return launch_bias<DQK, DV, NORM_SIGMOID, CAUSAL>(p, dt, s);
    case NORM_ABSSUM: return launch_bias<DQK, DV, NORM_ABSSUM, CAUSAL>(p, dt, s);
    case NORM_ABS_OF_SUM: return launch_bias<DQK, DV, NORM_ABS_OF_SUM, CAUSAL>(p, dt, s);
    case NORM_NONE: return launch_bias<DQK, DV, NORM_NONE, CAUSAL>(p, dt, s);
    case BWD_NORM_NONE_RELU: return launch_bias<DQK, DV, BWD_NORM_NONE_RELU, CAUSAL>(p, dt, s);
  }
  return hipErrorInvalidValue;
}
template <int DQK, int DV>
hipError_t launch_dims(const BwdParams& p, const DecayTable& dt, int norm, int causal, hipStream_t s) {
  return causal ? launch_mask<DQK, DV, true>(p, dt, norm, s) : launch_mask<DQK, DV, false>(p, dt, norm, s);
}

}  // namespace
}  // namespace ae
