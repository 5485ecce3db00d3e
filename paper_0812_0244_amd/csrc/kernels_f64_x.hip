// Axis-3 passes (theta, assembly, the u probe) of the FP64 evaluation, every split
// class (see kernels.hpp).
#include "kernels.hpp"

namespace vdwnl {

hipError_t launch_x_f64(int kind, int cls, const LaunchArgs &a) { return launch_x<double>(kind, cls, a); }

}  // namespace vdwnl
