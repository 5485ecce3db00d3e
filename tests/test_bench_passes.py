"""The benchmark's record of the passes (host only): the passes that launch
kernels, and the bytes that each moves."""
import bench

SPECTRAL = ["x_deriv", "y_deriv", "z_deriv", "x_theta", "y_20f", "z_main", "y_20i", "x_assemble", "x_div", "y_div",
            "z_div", "reduce"]
STENCILS = ["fd_grad", "x_theta", "y_20f", "z_main", "y_20i", "x_assemble", "fd_div", "reduce"]


def test_passes_without_a_launch_are_left_out():
    t = {k: (1.0, 1) for k in SPECTRAL}
    assert list(bench.own_launches(t)) == [k for k in SPECTRAL if k not in ("y_deriv", "z_deriv", "reduce")]
    assert list(bench.own_launches(t, general=True)) == [k for k in SPECTRAL if k not in ("y_deriv", "reduce")]
    assert list(bench.own_launches({k: (1.0, 1) for k in STENCILS})) == STENCILS[:-1]


def test_pass_bytes_cover_merged_launches():
    """n in and grad n out for three directions; v_loc, q and v, per axis or (short
    edges) in one pass."""
    shape, s = (48, 50, 60), 4
    N = 48 * 50 * 60
    assert bench.pass_bytes("x_deriv", [shape], s) == 6 * N * s
    assert sum(bench.pass_bytes(k, [shape], s) for k in ("x_div", "y_div", "z_div")) == 9 * N * s
    small = (32, 24, 30)
    assert sum(bench.pass_bytes(k, [small], s) for k in ("x_div", "y_div", "z_div")) == 5 * 32 * 24 * 30 * s
