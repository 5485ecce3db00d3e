// Axis-2 passes of the 20 spectra and the one-axis derivatives of the FP32
// evaluation, every split class (see kernels.hpp).
#include "kernels.hpp"

namespace vdwnl {

hipError_t launch_y_f32(int kind, int cls, const LaunchArgs &a) {
    if (kind == KY_20F) return launch_y20<float, -1>(cls, a);
    if (kind == KY_20I) return launch_y20<float, 1>(cls, a);
    return launch_deriv<float>(kind, cls, a);
}

}  // namespace vdwnl
