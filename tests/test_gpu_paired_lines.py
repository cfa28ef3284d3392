"""The z pass that transforms two lines of one fixed end in one FFT: fields whose x modes differ by
their whole magnitude.  The reference is the Green solve by its defining sums in extended precision.

Tolerance 16 units of roundoff relative to the solution in the 2-norm (six transforms of a few
roundings each): the x and y transforms of these fields are exact, so nothing else is in it.  A
rounding of one line of a pair that reached the other would count by the ratio of their symbols,
up to 1e4 between the rough modes and the mean."""
import numpy as np
import pytest

from test_gpu_parity import _lib

pytestmark = pytest.mark.gpu

LD = np.longdouble
PI = LD("3.14159265358979323846264338327950288")


def _dct1(n):
    j = np.arange(n + 1)
    w = np.where((j == 0) | (j == n), 1, 2).astype(LD)
    B = np.cos(PI * (np.outer(j, j) % (2 * n)).astype(LD) / n) * w[None, :]
    s, q = np.sin(PI * j / n / 2) ** 2, np.cos(PI * j / n / 2) ** 2
    q[-1] = 0
    return B, B / (2 * n), s, q


def _dst3(n):
    m, j = np.arange(n), np.arange(n + 1)
    S = np.sin(PI * (np.outer(2 * m + 1, j) % (4 * n)).astype(LD) / (2 * n))
    w = np.where(j == n, 1, 2).astype(LD)
    h = PI * (m + LD(0.5)) / n / 2
    return S * w[None, :], S.T / n, np.sin(h) ** 2, np.cos(h) ** 2


def _green(x, n, lam, mu):
    """Nodes on z = 0 held, free elsewhere."""
    fx, ix, sx, qx = _dct1(n[0])
    fy, iy, sy, qy = _dct1(n[1])
    fz, iz, sz, qz = _dst3(n[2])
    SZ, QZ, SY, QY, SX, QX = sz[:, None, None], qz[:, None, None], sy[:, None], qy[:, None], sx, qx
    out = []
    for c in range(3):
        a = [LD(2 * mu + (lam if J == c else 0)) for J in range(3)]
        M = 4 * (a[0] * (SX * QY * QZ + QX * SY * SZ) + a[1] * (SY * QX * QZ + QY * SX * SZ)
                 + a[2] * (SZ * QX * QY + QZ * SX * SY))
        t = x[c].astype(LD)
        for f, i in ((fx, 2), (fy, 1), (fz, 0)):
            t = np.moveaxis(np.tensordot(f, t, (1, i)), 0, i)
        t = t / M
        for f, i in ((iz, 0), (iy, 1), (ix, 2)):
            t = np.moveaxis(np.tensordot(f, t, (1, i)), 0, i)
        out.append(t)
    return np.stack(out)


CASES = [((16, 16, L), "fp64") for L in (32, 48, 64, 96, 128, 256)] + [((64, 16, 128), "fp32"), ((64, 64, 64), "fp32")]


@pytest.mark.parametrize("top", [False, True])
@pytest.mark.parametrize("n,prec", CASES)
def test_rough_lines_do_not_reach_smooth_ones(n, prec, top):
    F = _lib()
    print(f"[paired lines] n={n} {prec} top={top}", flush=True)
    bc = np.zeros((3, 3, 2), np.int8)
    bc[:, 2, int(top)] = 1
    g = F.Solver(n, np.full(n[::-1], 1.25), np.full(n[::-1], 0.75), bc, r0_factor=1.0, precision=prec)
    # a comb along x without a mean: modes 8, 16, .. of 16 (or of 64, each eighth of them), no other
    comb = np.where(np.arange(n[0] + 1) % 4 == 0, 3.0, -1.0)
    z = np.arange(n[2] + 1)
    f = (16.0 + z)[:, None, None] * np.ones(n[1] + 1)[:, None] * comb
    f[0] = 0.0
    x = np.stack([f, 2.0 * f, -f])
    ref = _green(x, n, 1.25, 0.75)
    if top:
        u = g.stage_green(np.ascontiguousarray(x[:, ::-1]))[:, ::-1]
    else:
        u = g.stage_green(x)
    eps = 2.0 ** -53 if prec == "fp64" else 2.0 ** -24
    err = float(np.sqrt(((u - ref) ** 2).sum() / (ref ** 2).sum()))
    print(f"[paired lines] error {err / eps:.2f} units", flush=True)
    assert err <= 16 * eps
