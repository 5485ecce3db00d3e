"""Fused axis-1 tiles of one column and of two, on either contraction unit.

A tile holds a column pair where two columns fit the axis-1 budget (in FP64,
16 KB at most) and one column otherwise.  Both against the oracle on the same
(rounded) input at the bars of the parity tests, and their u spectra against
each other at the bars of the unit comparison; the two plans differ in their
number of tiles, so in the workspace they take.
"""
import numpy as np
import pytest

import workloads as W
from oracle import functional as F
from test_gpu_parity import check, fp32_input, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (shape, triclinic, precision, budget of one column, budget of two)
CASES = [((96, 96, 96), False, 32, 16384, 49152),
         ((20, 30, 18), False, 32, 4096, 49152),
         ((15, 8, 10), False, 32, 4096, 49152),
         ((20, 18, 24), True, 32, 4096, 49152),
         ((20, 30, 18), False, 64, 4096, 65536),
         ((20, 18, 24), True, 64, 4096, 65536)]


@pytest.mark.parametrize("shape,tilted,precision,one,two", CASES)
def test_one_and_two_columns_against_oracle(table, shape, tilted, precision, one, two):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0812_0244_amd import VdwNl
    from paper_0812_0244_amd.binding import CONTRACTION_MATRIX, CONTRACTION_VECTOR, STAGE_U_K
    rng = np.random.default_rng(77)
    if shape == (96, 96, 96):
        cell, n = W.gauss96().cell, W.gauss96().density()
    elif tilted:
        cell = W.triclinic_lattice(tuple(0.3 * s for s in shape), (85.0, 95.0, 80.0))
        n = W.density_on_lattice(shape, cell, W.random_atoms_lattice(rng, 4, cell))
    else:
        cell = tuple(0.3 * s for s in shape)
        n = W.density_on_grid(shape, cell, W.random_atoms(rng, 4, cell))
    if precision == 32:
        n = fp32_input(n)
    dt = torch.float64 if precision == 64 else torch.float32
    o = F.energy_potential(n, cell, table, return_parts=True)
    nt = torch.from_numpy(n).to("cuda", dt)
    units = (CONTRACTION_VECTOR, CONTRACTION_MATRIX) if precision == 32 and not tilted else (CONTRACTION_VECTOR,)
    bytes_, uks = {}, {}
    for budget in (one, two):
        for unit in units:
            lib = VdwNl(0)
            lib.set_grid(shape, cell, 0, precision)
            lib.set_kernel_table(table["qmesh"], table["qc"], 12, table["dk"], table["phi"], table["c_soft"])
            lib.set_tiling([65536, 65536, 65536, budget, 65536])
            lib.set_contraction(unit)
            v = torch.empty_like(nt)
            say("  %s %s budget %d unit %d" % (shape, "tilted" if tilted else "", budget, unit))
            ek, de = lib.energy_potential(nt.data_ptr(), v.data_ptr())
            check(dict(E_k=ek, dE=de, v=v.double().cpu().numpy()), o, precision)
            uk = torch.empty((shape[0], shape[1], shape[2] // 2 + 1, 20, 2), dtype=dt, device="cuda")
            lib.debug_stage(0, STAGE_U_K, uk.data_ptr())
            uks[budget, unit] = uk.double().cpu().numpy()
            bytes_[budget] = lib.info()[1]
    assert bytes_[one] > bytes_[two]                 # (one column a tile: more tiles)
    base = uks[one, CONTRACTION_VECTOR]
    for u in uks.values():
        assert np.abs(u - base).max() <= (2e-6 if precision == 32 else 1e-12) * np.abs(base).max()
