"""The vector form of the fused smoothing passes (whole z lines of 16-byte
vectors) at the edges of its tiles: lines of every vector count the hierarchy
rule allows, odd row remainders, a grid's whole plane in one workgroup, tiles of
8 to 24 rows, short, long and odd x chunks, and the lengths it leaves to the
scalar form (11 and 15 vertices in FP32, lines of over 64 vectors).

Each solve is compared with the same solve by the separate one-ring passes
(MLSGD_PRE2R=0, MLSGD_POST2=0, checked against the oracle elsewhere).  Both
preconditioners are the same up to rounding of the V-cycle's type, e = 2^-53 or
2^-24 times a few, so the iterates differ by about e times their error, far
below the solver tolerance; what remains is FP64 rounding of the solves, about
the condition number (under 1e5 here) times 1e-16 of the solution: 1e-11.  FP64
iteration counts agree; FP32 ones may differ by one at the exit test."""
import numpy as np
import pytest

from paper_2606_09291_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_09291_amd as m
    m.lib()
    return m


def _solve(mm, monkeypatch, flag, precision, n_list, tuning):
    monkeypatch.setenv("MLSGD_PRE2R", flag)
    monkeypatch.setenv("MLSGD_POST2", flag)
    prec = mm.FP64 if precision == "fp64" else mm.MIXED_FP32 if precision == "mixed" else mm.MIXED_BF16
    rtol = 1e-12 if max(n_list) < 129 else 1e-10   # above the FP64 residual floor
    ctx = mm.Context(mm.Problem(grid_n=[9, 17], y_d=inputs.target_sin(17), rtol=rtol,
                                precision=prec), use_tuned=False)
    if tuning:
        ctx.set_tuning(**tuning)
    ys, st = ctx.solve_sizes(n_list, level=6, first=3, f_value=1.0)
    ys = [y.cpu().numpy() for y in ys]
    ctx.close()
    assert st["nonconverged"] == 0
    return ys, st


@pytest.mark.parametrize("n_list,tuning", [
    ([11, 13, 15, 17, 21, 25, 29], {}),                 # one workgroup plane, dense coarse grids
    ([33, 41, 49, 57], {}),                             # whole planes and 12- to 24-row tiles
    ([65, 81, 97, 113], {}),                            # ragged last row tile
    ([129, 161, 257], {}),                              # 64 vectors a line; scalar form beyond
    ([17] * 300 + [33] * 40 + [15] * 5, {}),            # full batch: whole-line chunks
    ([17, 33, 65], {"xchunk": 9}),                      # odd chunks: full residual
    ([33, 65], {"xchunk": 40, "tile_y": 16}),
    ([33, 65], {"tile_y": 4}),                          # separate passes on 65, vector on 33
])
@pytest.mark.parametrize("precision", ["fp64", "mixed", "bf16"])
def test_vector_passes_equal_separate_passes(mm, monkeypatch, n_list, tuning, precision):
    print("vector passes", n_list[:8], tuning, precision, flush=True)
    if precision == "bf16" and max(n_list) > 129:
        n_list = [n for n in n_list if n <= 129]
    y0, s0 = _solve(mm, monkeypatch, "0", precision, n_list, tuning)
    y1, s1 = _solve(mm, monkeypatch, "1", precision, n_list, tuning)
    worst = max(np.linalg.norm(a - b) / np.linalg.norm(a) for a, b in zip(y0, y1))
    print("relative difference", worst, "iterations", s0["iterations"], s1["iterations"], flush=True)
    assert worst <= (1e-11 if max(n_list) < 129 else 1e-9)
    assert abs(s0["iterations"] - s1["iterations"]) <= (0 if precision == "fp64" else 1)
