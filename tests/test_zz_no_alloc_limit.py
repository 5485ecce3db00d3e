"""Plans at the size limit of vdwnl_energy_potential_noalloc: grids in
triclinic cells whose whole image (kernel rows packed) comes to 64 MiB, give
or take 0.1%, with the tile lists.  The static array holds them, and the result
equals the allocating call's bitwise."""
import numpy as np
import pytest

import workloads as W
from test_zz_no_alloc import _both, _check, _context

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape,precision,grad_mode", [((18, 15, 243), 64, 2), ((6, 54, 405), 32, 0)])
def test_noalloc_takes_plans_of_64_mib(table, shape, precision, grad_mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    h = 0.22
    a, b, c = (h * s for s in shape)
    lat = np.array([[a, 0.0, 0.0], [0.1 * a, b, 0.0], [0.05 * a, -0.1 * b, c]])
    d = W.density_on_lattice(shape, lat, W.random_atoms_lattice(np.random.default_rng(3), 2, lat))
    n = torch.from_numpy(d).to("cuda", torch.float64 if precision == 64 else torch.float32)
    _check(*_both(_context(shape, lat, table, precision, grad_mode), n), "%s fp%d" % (shape, precision))
