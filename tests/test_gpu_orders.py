"""A stored radix order changes nothing: neither the plan nor the results."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", [32, 64])
def test_orders_leave_plan_and_results(table, precision):
    """On a batch of thin grids whose axes take compile-time and run-time
    radices: after every order set, the planned device state is still there
    (the stage probe answers without another evaluation), and an evaluation
    equals the first one bitwise."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0812_0244_amd import VdwNl
    from paper_0812_0244_amd.binding import STAGE_THETA
    dt = torch.float64 if precision == 64 else torch.float32
    shapes = [(10, 12, 64), (128, 10, 12), (12, 96, 10), (9, 10, 27)]
    cells = [tuple(0.2 * x for x in s) for s in shapes]
    n = [torch.from_numpy(W.density_on_grid(s, c, W.random_atoms(np.random.default_rng(60 + i), 2, c))).to("cuda", dt)
         for i, (s, c) in enumerate(zip(shapes, cells))]
    lib = VdwNl(0)
    lib.set_grids(shapes, cells, 0, precision)
    lib.set_kernel_table(table["qmesh"], table["qc"], 12, table["dk"], table["phi"], table["c_soft"])

    def run():
        v = [torch.empty_like(x) for x in n]
        return lib.energy_potential_batched([x.data_ptr() for x in n], [x.data_ptr() for x in v]), v

    E0, v0 = run()
    theta = torch.empty((20,) + shapes[1], dtype=dt, device="cuda")
    for order in (5, 1):
        lib.set_radix_orders([order] * 5)
        assert set(lib.get_radix_orders().values()) == {order}
        lib.debug_stage(1, STAGE_THETA, theta.data_ptr())
        E, v = run()
        assert np.array_equal(E, E0) and all(torch.equal(a, b) for a, b in zip(v, v0))
