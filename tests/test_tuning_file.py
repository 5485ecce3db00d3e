"""Which entries of a tuning file a plan takes (host only: the file's keys are
formed from the grid list, the architecture, which is "host" without a device,
and the kernels' schedule)."""
import ctypes
import json

import numpy as np
import pytest

from paper_0812_0244_amd import binding as B

SHAPE, CELL = (20, 18, 24), (5.0, 4.5, 6.0)
DEFAULT = [65536] * 5


def _key(schedule):
    """The key of SHAPE in CELL, FP32, spectral gradient, 64 KB of LDS; the
    part behind the last slash is the FNV-1a hash of the plan's text."""
    text = "32/0/65536;%dx%dx%d@" % SHAPE
    text += "".join("%.17g," % x for x in np.diag(CELL).ravel())
    h = 1469598103934665603
    for ch in text.encode():
        h = ((h ^ ch) * 1099511628211) % 2 ** 64
    return "host%s/p32/g0/l65536/n1/%016x" % (schedule, h)


@pytest.mark.parametrize("schedule,taken", [("", False), ("/s1", False), ("/s2", True)])
def test_entries_of_other_tiles_are_not_taken(tmp_path, monkeypatch, schedule, taken):
    """An entry without a schedule number was tuned for tiles the kernels no
    longer have: the plan keeps its defaults.  One with the present number is
    taken."""
    path = tmp_path / "tuning.json"
    path.write_text('{\n  "%s": [16384, 16384, 16384, 16384, 16384, 0, 0, 0, 0, 0, 0]\n}\n' % _key(schedule))
    json.load(open(path))
    monkeypatch.setenv("VDWNL_TUNE_CACHE", str(path))
    lib = B.load_library()
    h = ctypes.c_void_p()
    assert lib.vdwnl_create(ctypes.byref(h), -1) == 0
    shape, cell = (ctypes.c_int32 * 3)(*SHAPE), (ctypes.c_double * 3)(*CELL)
    assert lib.vdwnl_set_grid(h, shape, cell, 0, 32) == 0
    out, unit = (ctypes.c_int64 * 5)(), ctypes.c_int32()
    assert lib.vdwnl_get_tiling(h, 5, out) == 5
    assert lib.vdwnl_get_schedule(h, 0, ctypes.byref(unit)) == 0
    assert list(out) == ([16384] * 5 if taken else DEFAULT)
    assert unit.value == (B.CONTRACTION_VECTOR if taken else B.CONTRACTION_MATRIX)
    lib.vdwnl_destroy(h)
