// Compiled instances: the MFMA kernel with run-time factor shapes and the factor in registers, fp32,
// contractions of up to 128.
#include "launch_pad.hpp"

namespace km {
template hipError_t launch_mfma_pad<float, 8>(const LaunchArgs&);
}  // namespace km
