"""Where the one-kernel cycle from 17^3 down gives way to the separate passes.

mid_rows decides by the workgroups it would take: one for a problem on 17^3, one
for nine problems with their top grid on 9^3 (host code, no GPU needed).  Around
each line of the rule, estimates through the kernel and through the level-by-level
path (MLSGD_VSMALL=0) agree to FP64 rounding of the solves: condition number (under
1e4 at these sizes) times 1e-16 with a margin of 10, as for the kernel's other
edges; FP64 iteration counts agree, FP32 ones may differ by one at the exit test."""
import ctypes
import os

import numpy as np
import pytest

from paper_2606_09291_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rule():
    path = os.path.join(ROOT, "paper_2606_09291_amd", "libmlsgd.so")
    if not os.path.exists(path):
        pytest.skip("libmlsgd.so not built")
    f = ctypes.CDLL(path)._ZN5mlsgd8mid_rowsEiii
    f.restype = ctypes.c_bool

    def rule(rows17, packs, elem):   # the same for any filling of the last pack
        got = {f(rows17, t, elem) for t in ([9 * packs - 8, 9 * packs] if packs else [0])}
        assert len(got) == 1
        return got.pop()

    assert rule(1, 0, 8) and rule(1024, 0, 8) and not rule(1025, 0, 8)
    assert rule(2, 254, 8) and not rule(2, 255, 8)
    assert not rule(127, 130, 8) and rule(128, 129, 8)
    assert rule(256, 256, 8) and not rule(256, 257, 8) and not rule(512, 1, 8)
    assert not rule(64, 8000, 8) and not rule(2, 1 << 20, 8)
    assert rule(2, 1278, 4) and not rule(2, 1279, 4)
    assert rule(1024, 256, 4) and not rule(1024, 257, 4) and not rule(1025, 0, 4)


@pytest.mark.gpu
@pytest.mark.parametrize("precision,M", [
    ("fp64", [2284, 2]), ("fp64", [2285, 2]),          # 256 and 257 workgroups
    ("fp64", [3328, 128]), ("fp64", [3329, 128]),      # 512 and 513
    ("mixed", [11500, 2]), ("mixed", [11501, 2])])     # 1280 and 1281
def test_estimates_around_the_lines(monkeypatch, precision, M):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_09291_amd as mm
    print("around the lines", precision, M, flush=True)
    yd = inputs.target_sin(17)
    u = inputs.control_xyz(17) + 15.0 * yd
    out = []
    for flag in ("0", "1"):
        monkeypatch.setenv("MLSGD_VSMALL", flag)
        ctx = mm.Context(mm.Problem(grid_n=[9, 17], y_d=yd, rtol=1e-12,
                                    precision=mm.FP64 if precision == "fp64" else mm.MIXED_FP32),
                         use_tuned=False)
        g, st = ctx.mlmc_gradient(u, M, first=[2, 2])
        out.append((g.cpu().numpy(), st))
        ctx.close()
        assert st["nonconverged"] == 0
    d = float(np.linalg.norm(out[1][0] - out[0][0]) / np.linalg.norm(out[0][0]))
    print("relative difference", d, flush=True)
    assert d <= 1e-11
    for key in ("iters_state", "iters_adjoint"):
        assert abs(out[0][1][key] - out[1][1][key]) <= (0 if precision == "fp64" else 1)
