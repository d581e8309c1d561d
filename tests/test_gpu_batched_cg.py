"""Unpreconditioned CG on grids above 17^3, and on 17^3 beside one: the batched
iteration with cached coefficients (grids up to 17^3 alone take one workgroup a
solve).

Single-level and two-level gradients against the oracle, host-driven and as graph
replays: both solve to rtol 1e-12, so gradients agree to the condition number of
the operator (under 1e4) times that, 1e-8.  With the step of x deferred into the
next matvec and without, the iterates are the same operations on the same
operands, one pass apart, so the bits are the same, also where an iteration limit
ends the loop with every step pending."""
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


def _estimates(mm, grid, M, graph=False, max_iters=500):
    import torch
    n = grid[-1]
    yd = inputs.target_sin(n)
    ctx = mm.Context(mm.Problem(grid_n=grid, y_d=yd, theta=1.0, solver=mm.SOLVER_CG, rtol=1e-12,
                                max_iters=max_iters), use_tuned=False)
    if graph:
        ctx.set_graph(True)
    u = torch.as_tensor(inputs.control_xyz(n) + 15.0 * yd, device="cuda:0").contiguous()
    out = []
    for r in range(3 if graph else 1):   # graph: capture, then two replays
        g, st = ctx.mlmc_gradient(u, M, first=[r * m for m in M], allow_noconv=True)
        torch.cuda.synchronize()
        out.append((g.cpu().numpy().copy(), st))
    ctx.close()
    return out


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("grid,M", [([33], [5]), ([17, 33], [6, 3])])
def test_gradient_matches_oracle(mm, orc, grid, M, graph):
    print("batched CG", grid, M, graph, flush=True)
    n = grid[-1]
    yd = inputs.target_sin(n)
    u = inputs.control_xyz(n) + 15.0 * yd
    pb = orc.make_problem(grid, theta=1.0, rtol=1e-14)
    for r, (g, st) in enumerate(_estimates(mm, grid, M, graph)):
        go, so = orc.mlmc_gradient(pb, None, u, yd, M, first=[r * m for m in M])
        err = float(np.linalg.norm(g - go) / np.linalg.norm(go))
        print("relative error", err, "iterations", st["iters_state"], flush=True)
        assert st["nonconverged"] == 0 and st["iters_state"] > 50
        assert err <= 1e-8
        assert abs(st["J"] - so["J"]) <= 1e-8 * abs(so["J"])


@pytest.mark.parametrize("grid,M", [([33], [5]), ([17, 33], [6, 3])])
@pytest.mark.parametrize("max_iters", [500, 7])
def test_deferred_step_is_bit_identical(mm, monkeypatch, grid, M, max_iters):
    print("batched CG, deferred step", grid, M, max_iters, flush=True)
    res = []
    for flag in ("0", "1"):
        monkeypatch.setenv("MLSGD_XDEFER", flag)
        res.append(_estimates(mm, grid, M, max_iters=max_iters)[0])
    (g0, s0), (g1, s1) = res
    assert np.array_equal(g0, g1)
    for key in ("J", "s", "iters_state", "iters_adjoint", "max_relres", "nonconverged"):
        assert s0[key] == s1[key], key
    assert (s1["iters_state"] == 7 and s1["nonconverged"] > 0) if max_iters == 7 else \
        s1["nonconverged"] == 0
