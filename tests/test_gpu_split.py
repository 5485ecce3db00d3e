"""Transform lengths of every class on every axis.

A length runs as two register DFTs (its most even split R1 R2) in a kernel
compiled for its class of largest radix (10, 16 or 27), or through the
run-time radix passes where it has no such split.  The lengths here are the
ends of each class, primes and prime powers (R1 = 1, unequal radices), odd
ones, and the first ones past the split lengths; the other two axes stay
short.  The stages against the oracle's and the transforms against numpy's, at
the bars of the stage tests, in orthorhombic and (axis 1, whose pass has a
variant for them) triclinic cells.
"""
import numpy as np
import pytest

import workloads as W
from oracle import functional as F
from test_gpu_stages import NQ, check_against_oracle, rel, say, stages

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LENS = {0: (4, 5, 27, 81, 100, 108, 125, 162, 200),
        1: (4, 5, 27, 100, 108, 125, 256, 243, 324, 405, 432, 512),
        2: (4, 5, 27, 81, 100, 108, 125, 256, 243, 324, 405)}
CASES = [(a, n, False) for a, ls in LENS.items() for n in ls] + [(0, n, True) for n in LENS[0]]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("axis,L,tilted", CASES)
def test_split_lengths(table, axis, L, tilted):
    shape = [6, 4]
    shape.insert(axis, L)
    shape = tuple(shape)
    rng = np.random.default_rng(500 + 3 * L + axis)
    if tilted:
        cell = W.triclinic_lattice(tuple(0.25 * s for s in shape), (85.0, 95.0, 80.0))
        n = W.density_on_lattice(shape, cell, W.random_atoms_lattice(rng, 2, cell))
    else:
        cell = tuple(0.2 * s for s in shape)      # max |G| = pi sqrt(3) / 0.2 = 27.2 < 32
        n = W.density_on_grid(shape, cell, W.random_atoms(rng, 2, cell))
    for precision in (64, 32):
        say("  axis %d length %d fp%d shape %s %s" % (axis + 1, L, precision, shape, "tilted" if tilted else ""))
        nin = n if precision == 64 else n.astype(np.float32).astype(np.float64)
        o = F.energy_potential(nin, cell, table, return_parts=True)
        g = stages([nin], [cell], table, precision)[0]
        check_against_oracle(g, o, precision, "%s" % (shape,))
        N = n.size
        ref_c = np.stack([np.fft.rfftn(g["theta"][a]) for a in range(NQ)]) / N
        ref_u = np.stack([np.fft.irfftn(g["uhat"][a], s=shape, axes=(0, 1, 2)) for a in range(NQ)]) * N
        bar = 1e-13 if precision == 64 else 2e-6
        assert rel(g["chat"], ref_c) <= bar and rel(g["u"], ref_u) <= bar
