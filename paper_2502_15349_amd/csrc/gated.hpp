// Recurrent pattern with per-token gates: what ae_attn.hip needs to know of gated_recurrent.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_kernel.hpp"  // DecayTable

namespace ae {
struct GatedParams {
  const __bf16* Q;          // [B, H_qk, L, D_qk]
  const __bf16* K;          // [B, H_qk, L, D_qk]
  const __bf16* V;          // [B, H_v, L, D_v] (H_v = H unless the backward pass swaps the roles of the operands)
  const float* log_decay;   // [B, H, L]: ln a_t <= 0; null: one constant decay per head, from the table passed beside
  const float* key_gate;    // [B, H, L] or null (ones): the factor g_t on the key -- or, with gate_on_output, on the
                            // output row of token t instead (the two never occur together)
  const float* h_in;        // [B, H, D_qk, D_v] fp32 or null (zero)
  float* h_out;             // the same layout, or null
  void* O;                  // [B, H, L, D_v] fp32, or bf16 if out_bf16
  int B, H, H_qk, L;
  float scale;
  int out_bf16;
  int H_v = 0;         // heads of V (0: H): H, or a divisor of it (contiguous groups of H / H_v heads read the same V head)
  int gate_on_output = 0;  // key_gate multiplies o_t, not k_t
  // Walk the tokens from the last to the first: the recurrence runs over tau = L - 1 - t, token tau's decay is
  // log_decay[t + 1] (0 for the last token of the sequence, which is the first of the walk).  Only the memory
  // addresses change.  This is the form the sums over later tokens of the backward pass take.
  int reverse = 0;
  // Segments: the walk of a (batch, head) cut into nseg pieces of seg_len tokens (a multiple of 64; the last may be
  // shorter), one workgroup each.  h_in / h_out are then [B, H, nseg, D_qk, D_v]: every segment starts from its
  // own slot and leaves its final state in its own slot -- unless h_out_last_only, where h_out is [B, H, D_qk, D_v]
  // and only the last segment writes.  nseg = 1: the whole sequence, the layouts above.
  int nseg = 1;
  int seg_len = 0;
  int h_out_last_only = 0;
  // state_only: no outputs -- only the state update is walked (O is not touched); seg_decay, if set, receives the
  // sum of the segment's log-decays, fp32 [B, H, nseg]
  int state_only = 0;
  // 2: a workgroup walks two consecutive value heads of one q/k head, whose tiles and scores they share (D_v = 64, an even
  // number of value heads per q/k head, H_v = H; in launch_gated_backward beside several heads of the first two walks only)
  int heads_per_workgroup = 1;
  float* seg_decay = nullptr;
  // part: only the tokens [seg_from, seg_to) of the walk, in nseg >= 1 segments; h_in holds in_slots states for a (batch, head), of which
  // segment i starts from the i-th, h_out (and seg_decay) out_slots (the pointers may stand at another slot than the first).
  // Kernels of their own: reading these fields cost the other launches 0.2 us each.
  int part = 0;
  int seg_from = 0, seg_to = 0, in_slots = 1, out_slots = 1;
};
// A walk's first segment in full (lead: whole rows of outputs, its final state) and the states of later ones (states: state_only),
// side by side in one launch.  The same constant decays for both.
hipError_t launch_gated_lead(const GatedParams& lead, const GatedParams& states, const DecayTable& dt, int dqk, int dv, hipStream_t s);
// In place on buf [B, H, nseg, D_qk x D_v]: slot 0 holds the state in front of the first segment, slot i > 0 what segment i - 1 adds to
// it (its final state from a zero start), seg_decay[i] that segment's decay; slot i becomes the state in front of segment i.
hipError_t launch_gated_chain_segments(float* buf, const float* seg_decay, int BH, int nseg, int state_elems, hipStream_t s);
// In place on buf [B, H, nseg, D_qk x D_v] (the segments' final states from a zero start, as a state_only walk
// leaves them): slot s becomes the state in front of segment s, given the state in front of the sequence (h_in,
// [B, H, D_qk x D_v], or null for zero) and the segments' decays.
hipError_t launch_gated_combine_segments(float* buf, const float* seg_decay, const float* h_in, int BH, int nseg, int state_elems,
                                         hipStream_t stream);
// Epilogue of the backward pass (see ae_gated_backward): per q/k head and token, over the value heads of its group,
//   dB[h, t] = q_t . dQu[h, t] - g[h, t] (k_t . X[h, t]),   dkey_gate[h, t] = k_t . X[h, t],
//   dQ[t] = sum_h dQu[h, t],   dK[t] = sum_h g[h, t] X[h, t]
// and then dlog_decay[h, t] = sum_{i >= t} dB[h, i].  dQu / X may be dQ / dK themselves where H = H_qk.
struct GatedBwdEpilogueParams {
  const __bf16* Q;      // [B, H_qk, L, D_qk]
  const __bf16* K;
  const float* dQu;     // [B, H, L, D_qk]: gradient of q per value head
  const float* X;       // [B, H, L, D_qk]: gradient of the gated key per value head
  const float* key_gate;  // [B, H, L] or null
  float* dQ;            // [B, H_qk, L, D_qk]
  float* dK;
  float* dkey_gate;     // [B, H, L] or null
  float* dB;            // [B, H, L] workspace
  float* dlog_decay;    // [B, H, L]
  int B, H, H_qk, L;
};
hipError_t launch_gated_backward_epilogue(const GatedBwdEpilogueParams& p, int dqk, hipStream_t stream);
// The same gradients where value heads share q/k heads, summed over `heads` of them (at most kGatedGroupHeads; the last part of
// a group may have fewer) inside the walks: part `i` of a q/k head takes heads [i * heads, (i + 1) * heads) of its group and
// leaves its sum in out [B, H_qk, parts, L, D_qk].  Forwards (reverse = 0; Q = dO, K = V, V = K, R = Q): the gradient of q, the
// key gate on the keys, dots[h, t] = q_t . (gradient of q by head h).  Backwards (Q = V, K = dO, V = Q, R = K): the gradient of
// k, x_h being that of head h in front of its gate: the sum of g x_h, dkey_gate[h, t] = k_t . x_h, dots[h, t] = g k_t . x_h.
constexpr int kGatedGroupHeads = 4;
struct GatedGroupParams {
  const __bf16* Q;         // [B, H, L, D_v]
  const __bf16* K;         // [B, H, L, D_v]
  const __bf16* V;         // [B, H_qk, L, D_qk]
  const __bf16* R;         // [B, H_qk, L, D_qk]
  const float* log_decay;  // [B, H, L]
  const float* key_gate;   // [B, H, L] or null
  float* out;
  float* dots;             // [B, H, L]
  float* dkey_gate;        // [B, H, L] or null
  int B, H, H_qk, L;
  float scale;
  int reverse, heads, parts;
};
bool gated_group_supported(int dqk, int dv);
// dQ, dK [B, H_qk, L, D_qk]: the sums of the parts; head_elems = L * D_qk, elems = B * H_qk * L * D_qk
hipError_t launch_gated_group_sum(const float* dq_parts, const float* dk_parts, float* dQ, float* dK, int parts, int64_t head_elems,
                                  int64_t elems, hipStream_t stream);
// dlog_decay[h, t] = sum_{i >= t} dB[h, i] - minus[h, i] (minus: null, or dlog_decay itself); launch_gated_backward_epilogue ends with it
hipError_t launch_gated_suffix_sum(const float* dB, const float* minus, float* dlog_decay, int BH, int L, hipStream_t stream);
bool gated_supported(int dqk, int dv);
// 64/64, one head per workgroup: two workgroups can share a compute unit, and a launch can see to it that they don't.  Sharing evens out
// the last round and covers the start and the end of a walk; where the rounds of one each are full (at least `fill` of their places
// taken) and the calls stream through memory, one each reads it better (us, shared / one each): 9 x 32 heads x 2048 102 / 120, 12 x
// 32 x 2048 111 / 119, 18 x 32 x 2048 184 / 188, 64 x 32 x 512 135 / 142, 16 x 32 x 1024 70 / 71; but 15 x 32 x 2048 133 / 128, 28 x 32 x 2048 264 /
// 247, 32 x 32 x 2048 278 / 260, 16 x 64 x 1024 141 / 137.  Backward (three walks' workgroups): 12 x 32 x 2048 406 / 439, 8 x 32 x 1024 124 / 134,
// 20 x 32 x 2048 687 / 703; 8 x 32 x 4096 549 / 544, 8192 1100 / 1078.
inline bool gated_one_each(int64_t workgroups, int64_t tokens, int64_t from = 1024, double fill = 0.85) {
  return tokens >= from && workgroups * tokens >= 900000 && workgroups >= fill * 256 * ((workgroups + 255) / 256);
}
inline bool gated_backward_one_each(int64_t workgroups, int64_t tokens) { return gated_one_each(workgroups, tokens, 4096, 0.95); }
// dt: log2 of the per-head decay, read only where p.log_decay is null
hipError_t launch_gated_recurrent(const GatedParams& p, const DecayTable& dt, int dqk, int dv, hipStream_t stream);
// The three walks of the backward pass (dims D_v / D_qk, D_v / D_qk, D_qk / D_v, all cut alike) in one launch; group: the first two
// take these instead, several heads each.  dqk, dv: those of the forward pass.
hipError_t launch_gated_backward(const GatedParams (&walk)[3], const GatedGroupParams* group, int dqk, int dv, hipStream_t stream);
}  // namespace ae
