"""Kernels that keep a whole small problem in one workgroup, at the edges of
their ranges.

The V-cycle and the full-multigrid start from 17^3 down (one workgroup per
problem, a wave for each problem whose top grid is 9^3) against the same solve
level by level (MLSGD_VSMALL=0, checked against the oracle elsewhere): one
problem, the largest batch that takes it and one more, 9^3 problems in and
around whole workgroups of nine, one and three smoothing steps.  Both
preconditioners are the same up to rounding, so what remains is FP64 rounding of
the solves: condition number (under 1e4 at these sizes) times 1e-16 with a
margin of 10, and for gradients, which weight whole fields, the same.  FP64
iteration counts agree; FP32 ones may differ by one at the exit test.

Unpreconditioned CG on grids up to 17^3 against the level-by-level path
(MLSGD_CACHE64=0 leaves it no coefficient cache) at every size class, with the
oracle for the solution: both stop at a true relative residual of 1e-12, so the
solutions differ from the exact one by at most the condition number of the
diagonally unscaled operator (under 1e4) times that, 1e-8.  The dots' summation
order differs, so counts may differ by two in a hundred; at an iteration limit
they are the limit, and the iterates agree as far.

The matvec of all grid sizes in one launch against a launch per size (event
timing of the matvec keeps those): the same tiles and sums, so the same bits."""
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


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _prec(mm, precision):
    return {"fp64": mm.FP64, "mixed": mm.MIXED_FP32, "bf16": mm.MIXED_BF16}[precision]


@pytest.mark.parametrize("precision", ["fp64", "mixed", "bf16"])
@pytest.mark.parametrize("n_list,nu", [([17], 2), ([17] * 1024, 2), ([17] * 1025, 2),
                                       ([17, 17, 33, 65], 2), ([17, 33], 1), ([17, 33], 3)])
def test_cycle_from_17(mm, monkeypatch, n_list, nu, precision):
    print("cycle from 17", len(n_list), nu, precision, flush=True)
    monkeypatch.setenv("MLSGD_NU", str(nu))
    out = []
    for flag in ("0", "1"):
        monkeypatch.setenv("MLSGD_VSMALL", flag)
        ctx = mm.Context(mm.Problem(grid_n=[9, 17], y_d=inputs.target_sin(17), rtol=1e-12,
                                    precision=_prec(mm, precision)), use_tuned=False)
        ys, st = ctx.solve_sizes(n_list, level=6, first=3, f_value=1.0)
        out.append(([y.cpu().numpy() for y in ys], st))
        ctx.close()
        assert st["nonconverged"] == 0
    worst = max(_rel(b, a) for a, b in zip(out[0][0], out[1][0]))
    its = [o[1]["iterations"] for o in out]
    print("relative difference", worst, "iterations", its, flush=True)
    assert worst <= 1e-11
    assert abs(its[0] - its[1]) <= (0 if precision == "fp64" else 1)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("M", [[2, 2, 2], [7, 2, 2], [8, 2, 2], [500, 90, 11]])
def test_cycle_from_17_with_9_tops(mm, monkeypatch, M, precision):
    print("cycle from 17, tops on 9", M, precision, flush=True)
    yd = inputs.target_sin(33)
    u = inputs.control_xyz(33) + 15.0 * yd
    out = []
    for flag in ("0", "1"):
        monkeypatch.setenv("MLSGD_VSMALL", flag)
        ctx = mm.Context(mm.Problem(grid_n=[9, 17, 33], y_d=yd, rtol=1e-12,
                                    precision=_prec(mm, precision)), use_tuned=False)
        g, st = ctx.mlmc_gradient(u, M, first=[2] * 3)
        out.append((g.cpu().numpy(), st))
        ctx.close()
        assert st["nonconverged"] == 0
    d = _rel(out[1][0], out[0][0])
    print("relative difference", d, flush=True)
    assert d <= 1e-11
    for key in ("iters_state", "iters_adjoint"):
        assert abs(out[0][1][key] - out[1][1][key]) <= (0 if precision == "fp64" else 1)


@pytest.mark.parametrize("max_iters", [2000, 7])
@pytest.mark.parametrize("count", [1, 300])
def test_small_cg(mm, orc, monkeypatch, count, max_iters):
    print("small CG", count, max_iters, flush=True)
    for n in (5, 7, 9, 11, 13, 15, 17):
        out = []
        for cache in ("0", "1"):
            monkeypatch.setenv("MLSGD_CACHE64", cache)
            ctx = mm.Context(mm.Problem(grid_n=[9, 17], y_d=inputs.target_sin(17), rtol=1e-12,
                                        max_iters=max_iters, solver=mm.SOLVER_CG),
                             use_tuned=False)
            ys, st = ctx.solve_sizes([n] * count, level=4, first=1, f_value=1.0, allow_noconv=True)
            out.append(([y.cpu().numpy() for y in ys], st))
            ctx.close()
        its = [o[1]["iterations"] for o in out]
        worst = max(_rel(b, a) for a, b in zip(out[0][0], out[1][0]))
        print(n, "iterations", its, "relative difference", worst, flush=True)
        assert out[0][1]["nonconverged"] == out[1][1]["nonconverged"]
        assert abs(its[0] - its[1]) <= 2 and max(its) <= max_iters
        assert worst <= 1e-8
        if out[1][1]["nonconverged"]:
            assert max_iters == 7 and its == [7, 7]
            continue
        assert out[1][1]["max_relres"] <= 1e-12
        rhs = inputs.constant(n, 1.0)
        rhs[0] = rhs[-1] = 0
        rhs[:, 0] = rhs[:, -1] = 0
        rhs[:, :, 0] = rhs[:, :, -1] = 0
        for m in (0, count - 1):
            yo, _, _ = orc.solve(n, orc.kl_coeffs(0, 4, 1 + m, 4, 1.0), rhs, rtol=1e-14)
            assert _rel(out[1][0][m], yo) <= 1e-8


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("grid,M,tuning", [
    ([9, 17], [2, 2], {}), ([9, 17, 33, 65], [19, 7, 3, 2], {}),
    ([17, 33, 65, 129], [33, 9, 3, 2], {"xchunk": 9}), ([33, 65], [3, 2], {"tile_y": 16})])
def test_groups_in_one_launch(mm, grid, M, tuning, precision):
    print("groups in one launch", grid, M, tuning, precision, flush=True)
    yd = inputs.target_sin(grid[-1])
    u = inputs.control_xyz(grid[-1]) + 15.0 * yd
    out = []
    for timed in (False, True):
        ctx = mm.Context(mm.Problem(grid_n=grid, y_d=yd, rtol=1e-11,
                                    precision=_prec(mm, precision)), use_tuned=False)
        if tuning:
            ctx.set_tuning(**tuning)
        if timed:
            ctx.kernel_timing(4, 65)
        g, st = ctx.mlmc_gradient(u, M)
        out.append((g.cpu().numpy(), st))
        ctx.close()
    assert bool(np.array_equal(out[0][0], out[1][0]))
    assert out[0][1]["J"] == out[1][1]["J"]
