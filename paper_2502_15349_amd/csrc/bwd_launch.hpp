// Launch templates of the backward kernels, shared by the per-head-dim instantiation files
// (attn_bwd_<D_qk>_<D_v>.hip), each of which defines one launch_backward_<D_qk>_<D_v>().
#pragma once
#include <algorithm>

#include "bwd.hpp"

namespace ae {
namespace {

// One wavefront per 32 own rows where two workgroups of it fit a CU (64/64, and the query side of 128/128 without a bias
// tensor), a pair of wavefronts elsewhere (the measurements stand at bwd_pair_walk).  64/64 with a bias tensor has
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
// 64 418 / 447, 128 448 / 469, 200 518 / 511, 256 502 / 509; 192/128 64 491 / 536, 128 540 / 565, 200 642 / 613, 256 622 / 618;
// 128/256 64 600 / 609, 96 662 / 631.  Causal without a window, 8 x 64 heads: 128/128 64 rows 36.4 / 38.6, 100 53.9 / 55.5, 128 60.5 /
// 64.0; 192/128 45.6 / 47.8, 67.9 / 74.7, 75.5 / 87.6; 128/256 64 rows 51.1 / 53.0 (100 rows 4 x 24 heads 26.9 / 25.3).
constexpr int64_t short_window(int dqk, int dv) { return dv == 256 ? 64 : dqk == 192 ? 160 : 256; }
constexpr int64_t short_walk(int dv) { return dv == 256 ? 64 : 128; }
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
      return window ? window * heads <= short_window(DQK, DV) : rows * heads <= short_walk(DV);
    };
    if constexpr (DQK == 128 && DV == 128 && !BIAS) {
      const bool short_key = CAUSAL && is_short(p.L_q, p.g);
      const bool both = CAUSAL ? key_wgs <= (p.g == 1 ? 48 : 32) : key_wgs <= 24 || workgroups <= 64;
      if constexpr (CAUSAL)
        if (short_key) return launch_sides<K1, Q1>(p, dt, s, both);
      return launch_sides<K2, Q1>(p, dt, s, both);
    } else {
      if constexpr (CAUSAL && (!BIAS || DQK == 128))
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
