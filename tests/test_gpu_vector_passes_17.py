"""The vector smoothing passes on 17^3 (lines of 8 or 4 vectors, a whole plane in
less than two waves), with the one-kernel cycles off in both legs: by default they
take 17^3 up to some thousand problems.

Compared with the separate one-ring passes (MLSGD_PRE2R=0, MLSGD_POST2=0, checked
against the oracle elsewhere): both preconditioners are the same up to rounding of
the V-cycle's type, so what remains is FP64 rounding of the solves, about the
condition number (under 1e5) times 1e-16 of the solution: 1e-11.  FP64 iteration
counts agree; FP32 ones may differ by one at the exit test."""
import numpy as np
import pytest

from paper_2606_09291_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 2, 40, 300, 3000])
@pytest.mark.parametrize("precision", ["fp64", "mixed", "bf16"])
def test_17(monkeypatch, precision, count):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_09291_amd as mm
    print("vector passes on 17", precision, count, flush=True)
    monkeypatch.setenv("MLSGD_VSMALL", "0")
    prec = {"fp64": mm.FP64, "mixed": mm.MIXED_FP32, "bf16": mm.MIXED_BF16}[precision]
    out = []
    for flag in ("0", "1"):
        monkeypatch.setenv("MLSGD_PRE2R", flag)
        monkeypatch.setenv("MLSGD_POST2", flag)
        ctx = mm.Context(mm.Problem(grid_n=[9, 17], y_d=inputs.target_sin(17), rtol=1e-12,
                                    precision=prec), use_tuned=False)
        ctx.kernel_timing(3, 17)
        ys, st = ctx.solve_sizes([17] * count, level=6, first=3, f_value=1.0)
        launches = ctx.kernel_timing(0, 0)["launches"]
        out.append((np.stack([y.cpu().numpy() for y in ys]), st))
        ctx.close()
        assert st["nonconverged"] == 0
        assert (launches > 0) == (flag == "1")   # the fused passes run in the second leg
    y0, y1 = out[0][0].reshape(count, -1), out[1][0].reshape(count, -1)
    worst = float((np.linalg.norm(y1 - y0, axis=1) / np.linalg.norm(y0, axis=1)).max())
    its = [o[1]["iterations"] for o in out]
    print("relative difference", worst, "iterations", its, flush=True)
    assert worst <= 1e-11
    assert abs(its[0] - its[1]) <= (0 if precision == "fp64" else 1)
