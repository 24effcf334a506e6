// Backward kernel instantiations for D_qk = 192, D_v = 128 with the causal mask (a file of its own for the sake of build time).
#include "bwd_launch.hpp"

namespace ae {
hipError_t launch_backward_192_128_causal(const BwdParams& p, const DecayTable& dt, int norm, hipStream_t stream) {
  return launch_mask<192, 128, true>(p, dt, norm, stream);
}
}  // namespace ae
