// Compiled instances: the MFMA kernel with run-time factor shapes and a slice per lane, fp32, chunks of 7 vectors.
#include "launch_lane.hpp"

namespace km {
template hipError_t launch_mfma_lane<7>(const LaunchArgs&);
}  // namespace km
