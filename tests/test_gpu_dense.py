"""Transforms as matrix products (axis lengths without a compile-time FFT, periodic axes): the Green
stage against the oracle at the edges of the 16-wide tiles and of the 8-deep steps, up to the
longest line they take (256 nodes), on every axis, with random boundary tables (all four DTT
types), periodic axes of even and odd length, and grids with one and with two line tiles per
block.  Tolerances as in test_gpu_parity.py: FP64 1e-12, FP32 3e-5."""
import numpy as np
import pytest

from oracle.solver import Solver as OSolver
from test_gpu_parity import _lib

pytestmark = pytest.mark.gpu

CASES = [((14, 15, 21), None), ((22, 33, 39), None), ((40, 42, 65), None), ((250, 3, 5), None), ((4, 252, 3), None),
         ((3, 5, 250), None), ((256, 4, 3), 0), ((5, 35, 3), 1), ((3, 4, 48), 2), ((26, 110, 104), None),
         ((110, 26, 104), None), ((110, 104, 26), None), ((16, 13, 32), None)]


@pytest.mark.parametrize("idx", range(len(CASES)))
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_green_as_matrix_products(idx, prec):
    F = _lib()
    n, per = CASES[idx]
    print(f"[dense green] n={n} periodic={per} prec={prec}", flush=True)
    rng = np.random.default_rng(700 + idx)
    lam = rng.uniform(0.3, 3, n[::-1]); mu = rng.uniform(0.2, 2, n[::-1])
    bc = rng.integers(0, 2, (3, 3, 2)).astype(np.int8)
    if per is not None:
        bc[:, per, :] = 2
    o = OSolver(n, lam, mu, bc, r0_factor=1.2)
    g = F.Solver(n, lam, mu, bc, r0_factor=1.2, precision=prec)
    x = rng.standard_normal(o.zeros().shape)
    x[o.plan.amask] = 0.0
    ref = o.green.apply(x)
    out = g.stage_green(x)
    tol = 1e-12 if prec == "fp64" else 3e-5
    assert np.abs(out - ref).max() <= tol * np.abs(ref).max()


def test_static_workspace_without_room_for_matrices():
    """A problem that fits the static workspace only without the transform matrices is bound to it
    all the same and runs its transforms as FFTs."""
    F = _lib()

    def need(n):
        h = F.fftc_create(n, F.FFTC_FP64)
        b = F.fftc_workspace_bytes(h)
        F.fftc_destroy(h)
        return b

    limit = F.FFTC_STATIC_WORKSPACE_BYTES
    n = (100, 91, 55)
    # one forward and inverse pair per axis: one transform type per axis here
    mats = sum(2 * 8 * ((v + 16) // 16) * 16 * ((v + 8) // 8 * 8) for v in n)
    assert need(n) - mats + 4096 <= limit < need(n)
    print(f"[dense static] n={n}", flush=True)
    rng = np.random.default_rng(900)
    lam = rng.uniform(0.5, 2, n[::-1]); mu = rng.uniform(0.5, 2, n[::-1])
    bc = np.zeros((3, 3, 2), np.int8)
    bc[:, 2, 0] = 1
    a = F.Solver(n, lam, mu, bc, precision="fp64")
    b = F.Solver(n, lam, mu, bc, precision="fp64", static_workspace=True)
    x = rng.standard_normal((3, n[2] + 1, n[1] + 1, n[0] + 1))
    x[:, 0] = 0.0
    p, q = a.stage_green(x), b.stage_green(x)
    assert np.abs(p - q).max() <= 1e-12 * np.abs(p).max()


PERIODIC = [((16, 100, 104), 0), ((70, 32, 75), 1), ((60, 60, 48), 2), ((64, 5, 3), 0), ((6, 64, 4), 1), ((3, 5, 64), 2),
            ((96, 3, 6), 0), ((7, 96, 3), 1), ((33, 4, 96), 2), ((128, 4, 3), 0), ((40, 128, 2), 1), ((5, 2, 128), 2),
            ((256, 2, 3), 0), ((3, 256, 4), 1), ((35, 3, 256), 2)]


@pytest.mark.parametrize("idx", range(len(PERIODIC)))
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_green_periodic_compile_time_lengths(idx, prec):
    """Periodic axes of every length with a compile-time FFT (16, 32 and 48 on grids large enough that
    they are not taken as matrix products), each axis; tolerances as above."""
    F = _lib()
    n, per = PERIODIC[idx]
    print(f"[periodic green] n={n} periodic={per} prec={prec}", flush=True)
    rng = np.random.default_rng(800 + idx)
    lam = rng.uniform(0.3, 3, n[::-1]); mu = rng.uniform(0.2, 2, n[::-1])
    bc = rng.integers(0, 2, (3, 3, 2)).astype(np.int8)
    bc[:, per, :] = 2
    o = OSolver(n, lam, mu, bc, r0_factor=1.2)
    g = F.Solver(n, lam, mu, bc, r0_factor=1.2, precision=prec)
    x = rng.standard_normal(o.zeros().shape)
    x[o.plan.amask] = 0.0
    ref = o.green.apply(x)
    out = g.stage_green(x)
    tol = 1e-12 if prec == "fp64" else 3e-5
    assert np.abs(out - ref).max() <= tol * np.abs(ref).max()


PLANES = [((16, 16, 16), None), ((14, 15, 16), None), ((16, 14, 15), None), ((32, 30, 33), None), ((15, 48, 48), None),
          ((64, 64, 48), None), ((48, 39, 50), None), ((5, 2, 2), None), ((2, 65, 2), None), ((6, 2, 180), None),
          ((260, 14, 15), None), ((16, 16, 14), 1), ((14, 15, 16), 2), ((16, 13, 14), 0), ((96, 24, 22), None)]


@pytest.mark.parametrize("idx", range(len(PLANES)))
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_green_on_planes(idx, prec):
    """Small (y, z) planes, whose transforms between the x passes are one launch: edges of the 16-wide
    tiles, one and two line tiles per unit, both kinds of x pass next to it (and one that it is not
    taken with), planes of two nodes, periodic axes.  Tolerances as above."""
    F = _lib()
    n, per = PLANES[idx]
    print(f"[plane green] n={n} periodic={per} prec={prec}", flush=True)
    rng = np.random.default_rng(1100 + idx)
    lam = rng.uniform(0.3, 3, n[::-1]); mu = rng.uniform(0.2, 2, n[::-1])
    bc = rng.integers(0, 2, (3, 3, 2)).astype(np.int8)
    if per is not None:
        bc[:, per, :] = 2
    o = OSolver(n, lam, mu, bc, r0_factor=1.2)
    g = F.Solver(n, lam, mu, bc, r0_factor=1.2, precision=prec)
    x = rng.standard_normal(o.zeros().shape)
    x[o.plan.amask] = 0.0
    ref = o.green.apply(x)
    out = g.stage_green(x)
    tol = 1e-12 if prec == "fp64" else 3e-5
    assert np.abs(out - ref).max() <= tol * np.abs(ref).max()


QUARTER = [((18, 22, 16), 0), ((70, 54, 48), 1), ((130, 33, 32), 0), ((3, 5, 64), 1), ((65, 3, 64), 0), ((18, 4, 96), 0),
           ((64, 2, 96), 1), ((33, 3, 128), 0), ((5, 2, 128), 1), ((15, 3, 256), 0), ((32, 2, 256), 1)]


@pytest.mark.parametrize("idx", range(len(QUARTER)))
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_green_quarter_wave_z_lines(idx, prec):
    """z lines fixed at one end in every component (DCT3 or DST3), which share an FFT in pairs: each
    compile-time length, full and partial blocks of lines and a second line beyond the grid.
    Tolerances as above."""
    F = _lib()
    n, end = QUARTER[idx]
    print(f"[quarter green] n={n} fixed end={end} prec={prec}", flush=True)
    rng = np.random.default_rng(1200 + idx)
    lam = rng.uniform(0.3, 3, n[::-1]); mu = rng.uniform(0.2, 2, n[::-1])
    bc = rng.integers(0, 2, (3, 3, 2)).astype(np.int8)
    bc[:, 2, end], bc[:, 2, 1 - end] = 1, 0
    o = OSolver(n, lam, mu, bc, r0_factor=1.2)
    g = F.Solver(n, lam, mu, bc, r0_factor=1.2, precision=prec)
    x = rng.standard_normal(o.zeros().shape)
    x[o.plan.amask] = 0.0
    ref = o.green.apply(x)
    out = g.stage_green(x)
    tol = 1e-12 if prec == "fp64" else 3e-5
    assert np.abs(out - ref).max() <= tol * np.abs(ref).max()
