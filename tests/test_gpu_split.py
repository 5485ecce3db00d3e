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


@pytest.mark.parametrize("axis,L,tilted", [(a, n, t) for a, ls in LENS.items() for n in ls for t in (False, True)
                                           if not t or n in (4, 27, 108, 243, 512)])
def test_split_derivatives(table, axis, L, tilted):
    """grad n and the divergence along axes of every class, from the GPU's own
    q_c: grad against the oracle's spectral gradient, v_loc - v against the
    one-axis derivatives of q_c in numpy FFTs.  A spectral derivative, here or
    in numpy, rounds by its unit roundoff times the largest wave number times
    the largest value (in thin cells, where n is nearly uniform, far above
    |grad n|): bars of 1e-12 (FP64; some 4500 roundoffs) and 1e-6 (FP32; 16)
    of that scale plus the result's own."""
    from paper_0812_0244_amd import NonlocalCorrelation
    from paper_0812_0244_amd.binding import STAGE_GRAD
    shape = [6, 4] if L % 2 else [6, 5]          # (odd rows: unpaired last column)
    shape.insert(axis, L)
    if shape[0] * shape[1] % 2:
        shape = [x + 1 if x == 5 else x for x in shape]
    shape = tuple(shape)
    rng = np.random.default_rng(900 + 3 * L + axis)
    if tilted:
        cell = W.triclinic_lattice(tuple(0.25 * s for s in shape), (85.0, 95.0, 80.0))
        n = W.density_on_lattice(shape, cell, W.random_atoms_lattice(rng, 2, cell))
    else:
        cell = tuple(0.2 * s for s in shape)
        n = W.density_on_grid(shape, cell, W.random_atoms(rng, 2, cell))
    for precision in (64, 32):
        dt = torch.float64 if precision == 64 else torch.float32
        eng = NonlocalCorrelation(shape, cell, table, precision=precision, device=0)
        nt = torch.from_numpy(n).to("cuda", dt)
        say("  axis %d length %d fp%d shape %s %s" % (axis + 1, L, precision, shape, "tilted" if tilted else ""))
        # a view one element into a buffer: no access wider than an element is aligned
        vbuf = torch.empty(nt.numel() + 1, dtype=dt, device="cuda")
        v = vbuf[1:].view(shape)
        nbuf = torch.empty(nt.numel() + 1, dtype=dt, device="cuda")
        nbuf[1:].copy_(nt.reshape(-1))
        eng.lib.energy_potential(nt.data_ptr(), v.data_ptr())
        va = torch.empty_like(nt)
        eng.lib.energy_potential(nbuf[1:].data_ptr(), va.data_ptr())
        assert torch.equal(va, v)
        q = torch.empty((3,) + shape, dtype=dt, device="cuda")
        eng.lib.debug_field(0, 0, q.data_ptr())
        vl = torch.empty_like(nt)
        eng.lib.debug_field(0, 1, vl.data_ptr())
        g = torch.empty_like(q)
        eng.lib.debug_stage(0, STAGE_GRAD, g.data_ptr())
        bar = 1e-12 if precision == 64 else 1e-6
        ref = F.gradient(nt.double().cpu().numpy(), cell)
        kmax = np.pi * (5.0 if not tilted else 4.0 * 1.2)             # pi / spacing (the tilted cell's b_c: to 1.2)
        assert np.abs(g.double().cpu().numpy() - ref).max() <= bar * (np.abs(ref).max() + kmax * n.max())
        qd = q.double().cpu().numpy()
        div = 0.0
        for c in range(3):
            k = np.arange(shape[c] // 2 + 1) * (2 * np.pi / shape[c])
            if shape[c] % 2 == 0:
                k[-1] = 0.0
            k = k.reshape([-1 if a == c else 1 for a in range(3)])
            div = div + np.fft.irfft(1j * k * np.fft.rfft(qd[c], axis=c), n=shape[c], axis=c)
        ref_v = vl.double().cpu().numpy() - div
        scale = np.abs(ref_v).max() + np.pi * np.abs(qd).max(axis=(1, 2, 3)).sum()
        assert np.abs(v.double().cpu().numpy() - ref_v).max() <= bar * scale
