// Decoding shapes: what ae_attn.hip needs to know of attn_decode.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch.hpp"

namespace ae {
struct DecodeParams {
  const __bf16* Q;       // one row per (batch, q head): element strides qs[] = {batch, head}
  const __bf16* K;       // element strides ks[] = {batch, head, row}; rows 16-byte aligned
  const __bf16* V;
  float* ws_o;           // n_splits > 1: [n_splits, rows, D_v], normalised partial rows
  float* ws_lse;         // n_splits > 1: [n_splits, rows], their log-sum-exp without the bias (natural logarithm; -inf for a range without keys)
  void* O;               // n_splits == 1: the result, fp32 or (out_bf16) bf16, element strides os[] = {batch, head}
  float* stats;          // n_splits == 1, optional: [rows], the log-sum-exp
  int out_bf16;
  int64_t os[2];
  int64_t qs[2], ks[3], vs[3];
  int64_t rows;          // B * H_q
  int H_q, H_kv, g, L_k;  // g = H_q / H_kv
  int units;             // workgroups per set of q heads: B * H_kv * n_splits (set by launch_decode)
  int n_splits, split_keys;  // key range c: [c * split_keys, (c + 1) * split_keys)
  float c;               // scale * log2(e)
  float bias;            // constant bias of every score
};
// softmax with a plain or constant-bias modification, one query row per head, every key visible
bool decode_supported(int dqk, int dv);
hipError_t launch_decode(const DecodeParams& p, int dqk, int dv, hipStream_t stream);
}  // namespace ae
