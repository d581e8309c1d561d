"""The largest batches the allocation-free solve entry point accepts.

What the 64 MiB array holds follows from the arrays of a batch: per grid of the
hierarchy the solver rows, caches and reciprocal diagonals, five Krylov vectors
on the top grid, and per problem its keys, KL coefficients, scalars, slot lists
and partial sums, each array from a 256-byte boundary.  The largest batch by
that count is solved and equals the allocating entry point's result; one problem
more is refused, with the same count of bytes reported."""
import ctypes

import pytest

from paper_2606_09291_amd import inputs

pytestmark = pytest.mark.gpu

LIMIT = 64 << 20


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_09291_amd as m
    m.lib()
    return m


def _need(n, count, K, precision):
    """Bytes of a batch of `count` problems on n^3 (one partial slot each)."""
    off = 0

    def take(size):
        nonlocal off
        off = (off + 255) // 256 * 256 + size

    g = n
    while True:
        e = count * g ** 3
        widths = {"fp64": [8] * 5, "mixed": [8, 4, 4, 4, 4, 4, 8],
                  "bf16": [8, 4, 4, 4, 2, 4, 8]}[precision]
        for w in widths:
            take(w * e)
        if g == 3:
            break
        g = (g - 1) // 2 + 1
    for _ in range(5):
        take(8 * count * n ** 3)
    # level, sample, coefficients, Krylov scalars, slot offsets and counts, partials, phi, weight
    for w in (4, 8, 8 * K ** 3, 72, 4, 4, 8, 8, 8):
        take(w * count)
    return (off + 255) // 256 * 256 + 256


@pytest.mark.parametrize("precision,n,K,most", [
    ("fp64", 5, 4, 5731), ("fp64", 5, 1, 5989), ("mixed", 5, 4, 6045), ("mixed", 9, 4, 1091),
    ("bf16", 5, 4, 6215), ("fp64", 9, 4, 0)])
def test_largest_batch(mm, precision, n, K, most):
    import torch
    count = LIMIT // (70 * n ** 3)
    while _need(n, count, K, precision) > LIMIT:
        count -= 1
    assert most in (0, count)
    print("largest batch", precision, n, K, count, flush=True)
    prec = {"fp64": mm.FP64, "mixed": mm.MIXED_FP32, "bf16": mm.MIXED_BF16}[precision]
    yd = inputs.target_sin(n)
    u = inputs.control_xyz(n) + 20.0 * yd
    ctx = mm.Context(mm.Problem(grid_n=[n], y_d=yd, K=K, precision=prec, rtol=1e-12),
                     use_tuned=False)
    phi = torch.empty((count + 1,), dtype=torch.float64, device=ctx.device)
    st, need = ctx.solve_state_adjoint_noalloc(0, 0, 3, count, u, None, None, phi[:count])
    assert need == _need(n, count, K, precision) <= LIMIT
    _, _, ref, st_ref = ctx.solve_state_adjoint(0, 0, 3, count, u, want_y=False, want_p=False)
    torch.cuda.synchronize()
    assert st["nonconverged"] == 0 and st["iterations"] == st_ref["iterations"]
    assert float((phi[:count] - ref).abs().max() / ref.abs().max()) <= 1e-12
    uu = torch.as_tensor(u, device=ctx.device).contiguous()
    more = ctypes.c_int64(0)
    rc = ctx.lib.mlsgd_solve_state_adjoint_noalloc(
        ctx._h, 0, 0, 3, count + 1, ctypes.c_void_p(uu.data_ptr()), None, None,
        ctypes.c_void_p(phi.data_ptr()), None, ctypes.byref(more))
    assert rc == mm.MLSGD_EINVAL
    assert more.value == _need(n, count + 1, K, precision) > LIMIT
    ctx.close()
