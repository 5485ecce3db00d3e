// Axis-1 passes (the fused contraction pass, the gradient and divergence multipliers, the spectra probes) of the FP32 evaluation, every length class and radix order (see
// kernels.hpp).
#include "kernels.hpp"

namespace vdwnl {

hipError_t launch_z_f32(int kind, int lc, int var, const LaunchArgs &a) {
    if (kind == KZ_MAIN) return launch_zmain<float>(lc, 0, a);
    if (kind == KP_THETA_K) return launch_zmain<float>(lc, 1, a);
    if (kind == KP_U_K) return launch_zmain<float>(lc, 2, a);
    VDWNL_LC_VARIANTS(launch_z_lc, float, kind, lc, var, a)
}

}  // namespace vdwnl
