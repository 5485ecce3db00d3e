// The passes without a transform (finite-difference stencils, the theta
// probe) and the dispatch of every launch by precision and family (see
// kernels.hpp).
#include "kernels.hpp"

namespace vdwnl {

template <typename T>
static hipError_t launch_plain(int kind, const LaunchArgs &a) {
    if (a.ntiles == 0) return hipSuccess;    // (no LDS to raise)
    const dim3 grid(a.ntiles), block(a.threads);
    switch (kind) {
        case KF_GRAD: hipLaunchKernelGGL(k_fd_grad<T>, grid, block, 0, a.stream, a.insts, a.tiles); break;
        case KF_DIV: hipLaunchKernelGGL(k_fd_div<T>, grid, block, 0, a.stream, a.insts, a.tiles); break;
        case KP_THETA:
            hipLaunchKernelGGL(k_probe_theta<T>, grid, block, 0, a.stream, a.insts, a.tiles, a.cst, a.dst, a.target);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_kind(int kind, int lc, int precision, const LaunchArgs &a) {
    if (a.ntiles < 0) return hipErrorInvalidValue;
    const bool dp = precision == 64;
    switch (kind) {
        case KF_GRAD: case KF_DIV: case KP_THETA:
            return dp ? launch_plain<double>(kind, a) : launch_plain<float>(kind, a);
        case KX_THETA: case KX_ASSEMBLE: case KP_U:
            return dp ? launch_x_f64(kind, lc, a) : launch_x_f32(kind, lc, a);
        case KG_X: case KG_Y: case KG_Z: case KD_X: case KD_Y: case KD_Z: case KY_20F: case KY_20I:
            return dp ? launch_y_f64(kind, lc, a) : launch_y_f32(kind, lc, a);
        case KZ_MAIN: case KP_THETA_K: case KP_U_K:
            return dp ? launch_z_f64(kind, lc, a) : launch_z_f32(kind, lc, a);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_probe(int probe, int lc, int precision, const LaunchArgs &a, void *dst, int target) {
    static const int kinds[4] = {KP_THETA, KP_THETA_K, KP_U_K, KP_U};
    if (probe < 0 || probe > 3) return hipErrorInvalidValue;
    LaunchArgs b = a;
    b.dst = dst;
    b.target = target;
    return launch_kind(kinds[probe], lc, precision, b);
}

}  // namespace vdwnl
