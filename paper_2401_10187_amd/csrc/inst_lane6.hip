// Compiled instances: the MFMA kernel with run-time factor shapes and a slice per lane, fp32, chunks of 6 vectors.
#include "launch_lane.hpp"

namespace km {
template hipError_t launch_mfma_lane<6>(const LaunchArgs&);
}  // namespace km
