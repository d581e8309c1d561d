"""Tilings of the stencil kernels (host code of the library, no GPU): whatever
chunk length the environment holds, make_tiling and make_vtile return, with
chunks that cover the grid's planes; lengths below 8 stand for the default of
32.  Run in a process of its own with a time limit, so that a search for a chunk
that does not end fails the test."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROBE = r'''
import ctypes, sys
class VTile(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int) for k in ("R", "LZ", "full", "nty", "xchunk", "tiles", "PZ", "cyn", "czn", "lds")]
class Tiling(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int) for k in ("TY", "TZ", "nty", "ntz", "nxc", "xchunk", "tiles_per_row")]
L = ctypes.CDLL(sys.argv[1])
vt, mt = L._ZN5mlsgd10make_vtileEiiiii, L._ZN5mlsgd11make_tilingEiiii
vt.restype, mt.restype = VTile, Tiling
xchunk = int(sys.argv[2])
for n in (11, 17, 33, 49, 65, 129, 257):
    for rows in (0, 1, 40, 5000):
        t, d = mt(n, 8, xchunk, rows), mt(n, 8, 32, rows)
        assert t.xchunk >= 1 and t.nxc * t.xchunk >= n - 2 > (t.nxc - 1) * t.xchunk, (n, rows, t.xchunk)
        if xchunk < 8:
            assert t.xchunk == d.xchunk
        for elem in (4, 8):
            v, e = vt(n, elem, 8, xchunk, rows), vt(n, elem, 8, 32, rows)
            if v.R == 0:
                continue
            nxc = v.tiles // v.nty
            assert v.xchunk >= 1 and nxc * v.xchunk >= n - 2 > (nxc - 1) * v.xchunk, (n, rows, v.xchunk)
            if xchunk < 8:
                assert (v.xchunk, v.tiles) == (e.xchunk, e.tiles)
print("ok")
'''


@pytest.mark.parametrize("xchunk", [-(1 << 30), -8, 0, 1, 4, 7, 8, 9, 32, 40, 1024, 1 << 30])
def test_chunks_of_any_length(xchunk):
    lib = os.path.join(ROOT, "paper_2606_09291_amd", "libmlsgd.so")
    if not os.path.exists(lib):
        pytest.skip("libmlsgd.so not built")
    r = subprocess.run([sys.executable, "-c", PROBE, lib, str(xchunk)], capture_output=True,
                       text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stderr
