"""Device memory over re-plans that change the tiles (rows of the axis-3
tiles, columns of the fused axis-1 tiles), with graph replay: the context keeps
one workspace."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_replanning_other_tiles_keeps_one_workspace(table):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0812_0244_amd import VdwNl
    insts = W.batch_instances(64)[:16]
    lib = VdwNl(0)
    lib.set_grids([w.shape for w in insts], [w.cell for w in insts], 0, 32)
    lib.set_kernel_table(table["qmesh"], table["qc"], 12, table["dk"], table["phi"], table["c_soft"])
    n = [torch.from_numpy(w.density()).to("cuda", torch.float32) for w in insts]
    v = [torch.empty_like(x) for x in n]
    nptr, vptr = [x.data_ptr() for x in n], [x.data_ptr() for x in v]

    def free_bytes():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    E0 = lib.energy_potential_batched(nptr, vptr)          # (graph captured)
    ws, f0, seen = lib.info()[1], free_bytes(), set()
    for i in range(6):
        x, z = (65536, 65536) if i % 2 else (4096, 16384)
        lib.set_tiling([x, 65536, 65536, z, 65536])
        for _ in range(2):                                 # (capture, replay)
            E = lib.energy_potential_batched(nptr, vptr)
        seen.add(lib.info()[1])
        assert abs(E - E0).max() <= 1e-12 * abs(E0).max()  # (the grouping of the FP64 partial sums only)
    f1 = free_bytes()
    print("  plans of %s bytes; free memory %.2f -> %.2f GB" % (sorted(seen), f0 / 2 ** 30, f1 / 2 ** 30), flush=True)
    assert len(seen) == 2                                  # (the budgets gave other tiles)
    assert f0 - f1 < ws // 4
