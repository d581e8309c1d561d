"""The V-cycle and the full-multigrid start from 17^3 down in one kernel
(vcycle_mid), called by themselves, against the same cycle in numpy's extended
precision: harmonic faces 2 / (b_v + b_w) of the reciprocal coefficient b,
Chebyshev-weighted Jacobi steps down and in reverse order up, full weighting,
trilinear prolongation and the exact 3^3 solve.

Random coefficients: a value of z passes through about 60 roundings (five steps
of some twelve operations a grid, the reciprocals within one unit, u = 1.1e-16),
so z is within 60 u = 6.6e-15 at worst in relative L2; the bar is 1e-14.

Constant coefficient 1/a = c, checkerboard right-hand side: the cycle acts on
the finest grid alone (full weighting removes the checkerboard), where the faces
all carry the rounding of the one reciprocal 1 / (2 c), and z is proportional to
it.  The random magnitudes of b average the other roundings away over the
vertices (u / sqrt(3375)).  What may remain of <z - z_exact, z_exact> /
<z_exact, z_exact> is one u each for the face, the sum of six and the reciprocal
diagonal, to which z responds at most about twofold: 6 u, against which the bar
is 1e-15.  The c taken is one where a single Newton step from the hardware's
estimate leaves 2.1e-15 (two: at most u)."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LD = np.longdouble
SIZES = (17, 9, 5, 3)


class MidArgs(ctypes.Structure):
    _fields_ = ([(k, ctypes.c_int) for k in ("rows17", "rows9", "top17", "slots")] +
                [(k, ctypes.c_void_p) for k in ("b17", "b9", "c17", "c9", "c5", "c3", "x17", "x9")])


@pytest.fixture(scope="module")
def mm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_09291_amd as m
    m.lib()
    return m


def _omegas(deg, lo=0.15):
    a, b = 2.0 * lo, 2.0
    return [1.0 / (0.5 * (a + b) + 0.5 * (b - a) * np.cos(np.pi * (2 * j + 1) / (2 * deg)))
            for j in range(deg)]


class Cycle:
    """The cycle on grids of reciprocal coefficients b[n] (n^3 arrays)."""

    def __init__(self, b, om):
        self.om = [LD(w) for w in om]
        self.f, self.d = {}, {}
        for n, v in b.items():
            v = v.astype(LD)
            fx = LD(2) / (v[1:, 1:-1, 1:-1] + v[:-1, 1:-1, 1:-1])
            fy = LD(2) / (v[1:-1, 1:, 1:-1] + v[1:-1, :-1, 1:-1])
            fz = LD(2) / (v[1:-1, 1:-1, 1:] + v[1:-1, 1:-1, :-1])
            self.f[n] = (fx, fy, fz)
            self.d[n] = LD((n - 1) ** 2) * (fx[1:] + fx[:-1] + fy[:, 1:] + fy[:, :-1] +
                                            fz[..., 1:] + fz[..., :-1])

    def apply(self, n, x):
        fx, fy, fz = self.f[n]
        i = slice(1, -1)
        off = (fx[1:] * x[2:, i, i] + fx[:-1] * x[:-2, i, i] + fy[:, 1:] * x[i, 2:, i] +
               fy[:, :-1] * x[i, :-2, i] + fz[..., 1:] * x[i, i, 2:] + fz[..., :-1] * x[i, i, :-2])
        y = np.zeros_like(x)
        y[i, i, i] = self.d[n] * x[i, i, i] - LD((n - 1) ** 2) * off
        return y

    def smooth(self, n, x, b, om):
        i = slice(1, -1)
        for w in om:
            r = (b - self.apply(n, x))[i, i, i]
            x = x.copy()
            x[i, i, i] += w * r / self.d[n]
        return x

    @staticmethod
    def restrict(r):
        for ax in range(3):
            r = np.moveaxis(r, ax, 0)
            c = np.zeros((r.shape[0] // 2 + 1,) + r.shape[1:], dtype=LD)
            c[1:-1] = r[1:-3:2] / 4 + r[2:-2:2] / 2 + r[3:-1:2] / 4
            r = np.moveaxis(c, 0, ax)
        return r

    @staticmethod
    def prolong(c):
        for ax in range(3):
            c = np.moveaxis(c, ax, 0)
            f = np.zeros((2 * c.shape[0] - 1,) + c.shape[1:], dtype=LD)
            f[::2] = c
            f[1::2] = (c[1:] + c[:-1]) / 2
            c = np.moveaxis(f, 0, ax)
        return c

    def cycle(self, n, b, x=None):
        if x is None:
            x = np.zeros_like(b)
        if n == 3:
            x[1, 1, 1] = b[1, 1, 1] / self.d[3][0, 0, 0]
            return x
        x = self.smooth(n, x, b, self.om)
        m = n // 2 + 1
        x = x + self.prolong(self.cycle(m, self.restrict(b - self.apply(n, x))))
        return self.smooth(n, x, b, self.om[::-1])

    def start(self, b):
        bs = {17: b}
        for n in SIZES[1:]:
            bs[n] = self.restrict(bs[2 * n - 1])
        x = self.cycle(3, bs[3])
        for n in (5, 9, 17):
            x = self.cycle(n, bs[n], self.prolong(x))
        return x


def _run(mm, b, caches, om, start):
    """z of the problems b [rows, 17, 17, 17] by the kernel, in FP64."""
    import torch
    fn = mm.lib()._ZN5mlsgd10vcycle_midIdEEvPKdiiPKNS_6CgScalERKNS_7MidArgsIT_EEiPKiPdbP12ihipStream_t
    rows = b.shape[0]
    dev = [torch.as_tensor(np.ascontiguousarray(a), device="cuda:0") for a in [b] + caches]
    x17 = torch.zeros_like(dev[0])
    b9 = torch.zeros((rows, 9, 9, 9), dtype=torch.float64, device="cuda:0")
    x9 = torch.zeros_like(b9)
    ma = MidArgs(rows, rows, 0, 1, dev[0].data_ptr(), b9.data_ptr(),
                 *[d.data_ptr() for d in dev[1:]], x17.data_ptr(), x9.data_ptr())
    w = (ctypes.c_double * len(om))(*om)
    torch.cuda.synchronize()
    fn(w, ctypes.c_int(len(om)), ctypes.c_int(0), None, ctypes.byref(ma), ctypes.c_int(0), None,
       None, ctypes.c_bool(start), None)
    torch.cuda.synchronize()
    return x17.cpu().numpy()


@pytest.mark.parametrize("start", [False, True])
@pytest.mark.parametrize("deg", [1, 2, 3])
def test_random_coefficients(mm, deg, start):
    print("cycle from 17, random coefficients", deg, start, flush=True)
    rng = np.random.default_rng(deg)
    rows = 3
    caches = [np.exp(rng.standard_normal((rows, n, n, n))) for n in SIZES]
    b = np.zeros((rows, 17, 17, 17))
    b[:, 1:-1, 1:-1, 1:-1] = rng.standard_normal((rows, 15, 15, 15))
    om = _omegas(deg)
    z = _run(mm, b, caches, om, start)
    for m in range(rows):
        c = Cycle({n: caches[k][m] for k, n in enumerate(SIZES)}, om)
        ref = c.start(b[m].astype(LD)) if start else c.cycle(17, b[m].astype(LD))
        err = float(np.linalg.norm((z[m] - ref).astype(float)) / np.linalg.norm(ref.astype(float)))
        print("relative error", err, flush=True)
        assert err <= 1e-14


def test_reciprocals_of_17(mm):
    c = 0.99994564056396484   # a multiple of 2^-20
    rng = np.random.default_rng(7)
    k = np.arange(17)
    sign = (-1.0) ** (k[:, None, None] + k[None, :, None] + k[None, None, :])
    b = np.zeros((1, 17, 17, 17))
    b[0, 1:-1, 1:-1, 1:-1] = (sign * rng.uniform(0.9, 1.1, (17, 17, 17)))[1:-1, 1:-1, 1:-1]
    caches = [np.full((1, n, n, n), c) for n in SIZES]
    om = _omegas(2)
    z = _run(mm, b, caches, om, False)[0]
    ref = Cycle({n: np.full((n, n, n), c) for n in SIZES}, om).cycle(17, b[0].astype(LD))
    s = float(((z - ref) * ref).sum() / (ref * ref).sum())
    print("share of z off", s, flush=True)
    assert abs(s) <= 1e-15
