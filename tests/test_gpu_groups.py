"""The Krylov passes of all grid sizes in one launch (matvec, residual and its
norm, residual update, flush of pending steps) against a launch per size
(MLSGD_GROUPS=0): the same tiles and sums, so the same bits of gradients,
objectives, iteration counts and residuals.

Grids of every tile shape and line length class (9^3, 17^3, 33^3, 65^3 and the
129^3, 257^3 and 513^3 line walks), odd chunks, a tile height that takes a launch per
size for the matvec anyway, graph replays, and forced restarts, whose second
check and restarted right-hand sides go through the residuals that skip the
other problems."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_09291_amd as m
    m.lib()
    return m


CASES = [
    ("9..65", [9, 17, 33, 65], [19, 7, 3, 2], {}),
    ("9, 17, many", [9, 17], [700, 40], {}),
    ("17..129, odd chunks", [17, 33, 65, 129], [9, 5, 3, 2], {"xchunk": 9}),
    ("33, 65, tiles of 16", [33, 65], [3, 2], {"tile_y": 16}),
    ("9..33, restarts", [9, 17, 33], [16, 8, 4], {"restart": True}),
    ("9..33, graph with restarts", [9, 17, 33], [16, 8, 4], {"restart": True, "graph": True}),
    ("129, 257", [129, 257], [1, 1], {"rtol": 1e-9}),
    ("257, 513", [257, 513], [1, 1], {"rtol": 1e-9}),
]


def _estimate(mm, grid, M, precision, opts):
    import torch
    n = grid[-1]
    t = torch.linspace(0.0, 1.0, n, dtype=torch.float64, device="cuda:0")
    s = torch.sin(torch.pi * t)
    yd = s[:, None, None] * s[None, :, None] * s[None, None, :]
    u = 0.1 * t[:, None, None] * t[None, :, None] * t[None, None, :] + 15.0 * yd
    prec = mm.FP64 if precision == "fp64" else mm.MIXED_FP32
    ctx = mm.Context(mm.Problem(grid_n=grid, y_d=yd, theta=2.0, sigma2=2.0, precision=prec,
                                rtol=opts.get("rtol", 1e-12)), use_tuned=False)
    tuning = {k: opts[k] for k in ("xchunk", "tile_y") if k in opts}
    if tuning:
        ctx.set_tuning(**tuning)
    if opts.get("graph"):
        ctx.set_graph(True)
    out = []
    for r in range(3 if opts.get("graph") else 1):   # graph: capture, then two replays
        g, st = ctx.mlmc_gradient(u, M, first=[r * m for m in M])
        torch.cuda.synchronize()
        out.append((g.clone(), st))
    ctx.close()
    return out


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name,grid,M,opts", CASES, ids=[c[0] for c in CASES])
def test_one_launch_equals_a_launch_per_size(mm, monkeypatch, name, grid, M, opts, precision):
    import torch
    print("groups", name, precision, flush=True)
    if opts.get("restart"):
        monkeypatch.setenv("MLSGD_FORCE_RESTART", "1")
    res = []
    for flag in ("0", "1"):
        monkeypatch.setenv("MLSGD_GROUPS", flag)
        res.append(_estimate(mm, grid, M, precision, opts))
    for (g0, s0), (g1, s1) in zip(*res):
        assert torch.equal(g0, g1)
        for key in ("J", "s", "iters_state", "iters_adjoint", "max_relres", "nonconverged"):
            assert s0[key] == s1[key], key
        assert s1["nonconverged"] == 0
