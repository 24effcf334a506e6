// Backward kernel instantiations for D_qk = 192, D_v = 128.
#include "bwd_launch.hpp"

namespace ae {
hipError_t launch_backward_192_128_causal(const BwdParams&, const DecayTable&, int, hipStream_t);
hipError_t launch_backward_192_128(const BwdParams& p, const DecayTable& dt, int norm, int causal, hipStream_t stream) {
  return causal ? launch_backward_192_128_causal(p, dt, norm, stream) : launch_mask<192, 128, false>(p, dt, norm, stream);
}
}  // namespace ae
