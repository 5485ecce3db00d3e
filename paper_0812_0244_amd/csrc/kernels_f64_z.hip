// Fused axis-1 pass of the FP64 evaluation, every split class (see kernels.hpp).
#include "kernels.hpp"

namespace vdwnl {

hipError_t launch_z_f64(int kind, int cls, const LaunchArgs &a) {
    return launch_zmain<double>(cls, kind == KP_THETA_K ? 1 : kind == KP_U_K ? 2 : 0, a);
}

}  // namespace vdwnl
