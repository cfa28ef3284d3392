"""The marching residual pass of the FP32 form at the edges of its 31 x 7 node tiles: grids of a
little less than a tile, exactly one and a little more, two-voxel axes, segments of one and of
several planes, on every axis periodic, in small and finite strain, from u and incremental.  One
step from random fields through the stage entry against the oracle; tolerances as in
test_gpu_residual_form.py: 2e-5 with FP32 stresses, 2e-6 with FP64."""
import numpy as np
import pytest

import workloads as W
from oracle import tetra2
from oracle.solver import Solver as OSolver
from test_gpu_residual_form import _lib

pytestmark = pytest.mark.gpu

CASES = [((28, 5, 2), None), ((30, 6, 3), None), ((32, 7, 2), None), ((2, 2, 2), None), ((2, 14, 40), None),
         ((60, 2, 9), None), ((32, 7, 5), 0), ((30, 7, 5), 0), ((30, 7, 5), 1), ((32, 8, 2), 2), ((63, 13, 33), None)]


@pytest.mark.parametrize("idx", range(len(CASES)))
@pytest.mark.parametrize("form", ["fp32", "fp64_stress", "incremental", "finite_strain"])
def test_march_at_tile_edges(idx, form):
    F = _lib()
    n, per = CASES[idx]
    fs, f64, inc = form == "finite_strain", form == "fp64_stress", form == "incremental"
    print(f"[march] n={n} periodic={per} {form}", flush=True)
    rng = np.random.default_rng(1300 + idx)
    lam = rng.uniform(0.4, 2.5, n[::-1]); mu = rng.uniform(0.3, 1.8, n[::-1])
    bc = rng.integers(0, 2, (3, 3, 2)).astype(np.int8)
    bc[:, 0, 0] = W.BC_D          # no singular mode
    if per is not None:
        bc[:, per, :] = W.BC_P
        bc[:, (per + 1) % 3, 0] = W.BC_D
    o = OSolver(n, lam, mu, bc, r0_factor=1.3, finite_strain=fs)
    g = F.Solver(n, lam, mu, bc, r0_factor=1.3, precision="fp32", finite_strain=fs)
    A = o.plan.amask
    free = ~A

    def field(scale):
        f = rng.standard_normal(o.zeros().shape) * scale
        f[A] = 0.0
        return f

    u, delta, e, R_prev = field(2e-2), field(1e-3), field(2e-2), field(2e-2)
    pe = o.iterate_parts(u)["p"]
    p_prev = o.iterate_parts(u - delta)["p"] if inc else field(2e-2)
    k0d = -o.reference_term(tetra2.tet_gradients(delta, o.plan))
    p, R, dR, dY, sums = g.stage_residual_form(u, delta, e, p_prev, R_prev, 3, incremental=inc,
                                               fp64_stress=int(f64))
    tol = 2e-6 if f64 else 2e-5
    Re = pe + k0d - e
    dYe = pe - p_prev + k0d
    assert np.abs(p - pe).max() <= tol * np.abs(pe).max()
    assert abs(sums[0] - np.sum(pe[free] ** 2)) <= 10 * tol * np.sum(pe[free] ** 2)
    assert np.abs(R - Re)[free].max() <= tol * np.abs(Re).max()
    assert np.abs(dR - (Re - R_prev))[free].max() <= tol * np.abs(Re - R_prev).max()
    assert np.abs(dY - dYe)[free].max() <= tol * np.abs(dYe).max()


@pytest.mark.parametrize("idx", range(len(CASES) + 1))
@pytest.mark.parametrize("fs", [False, True])
def test_literal_march_at_tile_edges(idx, fs):
    """The FP64 pass of the literal form on the same tiles; the last grid's node plane has more tiles
    than a launch takes (node-centred kernel).  FP64 rounding: 1e-12."""
    F = _lib()
    n, per = (CASES + [((720, 720, 2), None)])[idx]
    if n[0] == 720 and fs:
        pytest.skip("the wide grid runs once")
    print(f"[march] n={n} periodic={per} fp64 finite_strain={fs}", flush=True)
    rng = np.random.default_rng(1400 + idx)
    lam = rng.uniform(0.4, 2.5, n[::-1]); mu = rng.uniform(0.3, 1.8, n[::-1])
    bc = rng.integers(0, 2, (3, 3, 2)).astype(np.int8)
    if per is not None:
        bc[:, per, :] = W.BC_P
    strong = [W.Strong(np.array([[1, 1, 1]]), np.array([1], np.int8), np.array([0.01]))]
    o = OSolver(n, lam, mu, bc, strong, r0_factor=1.3, finite_strain=fs)
    g = F.Solver(n, lam, mu, bc, strong, r0_factor=1.3, precision="fp64", finite_strain=fs)
    u = rng.standard_normal(o.zeros().shape) * 2e-2
    u[o.plan.amask] = 0.0
    parts = o.iterate_parts(u)
    p, pt, sums = g.stage_residual(u)
    assert np.abs(pt - parts["ptil"]).max() <= 1e-12 * np.abs(parts["ptil"]).max()
    assert np.abs(p - parts["p"]).max() <= 1e-12 * np.abs(parts["p"]).max()
    assert abs(sums[0] - parts["pnorm2"]) <= 1e-11 * parts["pnorm2"]
    assert abs(sums[1] - parts["sig2"]) <= 1e-11 * parts["sig2"]


@pytest.mark.parametrize("nx", [14, 16, 260])
@pytest.mark.parametrize("period", [2, 3])
def test_accelerated_iterates(nx, period):
    """The acceleration's ring of iterates under each kernel that combines them (matrix products,
    compile-time FFT, runtime-length FFT on x): 13 iterations of the FP64 form against the
    oracle's, every accelerating one among them (2 or 3 apart, so that a combination follows plain
    iterations of both parities).  1e-9: the iterates' sensitivity to rounding, as in
    test_gpu_parity.py."""
    F = _lib()
    n = (nx, 8, 6)
    print(f"[accelerated iterates] nx={nx} period={period}", flush=True)
    rng = np.random.default_rng(1500 + nx)
    lam = rng.uniform(0.4, 2.5, n[::-1]); mu = rng.uniform(0.3, 1.8, n[::-1])
    bc = np.zeros((3, 3, 2), np.int8)
    bc[:, 2, 0] = W.BC_D
    strong = [W.Strong(np.array([[3, 3, 6], [4, 3, 6]]), np.array([2, 2], np.int8), np.array([0.02, 0.02]))]
    o = OSolver(n, lam, mu, bc, strong, r0_factor=1.5).solve(tol=1e-14, period=period, max_iter=13)
    g = F.Solver(n, lam, mu, bc, strong, r0_factor=1.5, precision="fp64", tol=1e-14, period=period, max_iter=13)
    g.solve()
    u = g.u.cpu().numpy().reshape(o["u"].shape)
    assert np.linalg.norm(u - o["u"]) <= 1e-9 * np.linalg.norm(o["u"])


@pytest.mark.parametrize("size", [2, 7, 8, 9, 40, 63, 64])
@pytest.mark.parametrize("per", [None, 0, 2])
@pytest.mark.parametrize("fs", [False, True])
def test_projection_on_supports(size, per, fs):
    """proj_P of averages whose support fills part of a round of eight nodes, whole rounds and all
    eight rounds, on nodes anywhere in the grid (faces, edges, the seam of a periodic axis), against
    the oracle.  FP64 rounding: 1e-12."""
    F = _lib()
    n = (9, 8, 7)
    print(f"[supports] size={size} periodic={per} finite_strain={fs}", flush=True)
    rng = np.random.default_rng(1700 + size)
    lam = rng.uniform(0.4, 2.5, n[::-1]); mu = rng.uniform(0.3, 1.8, n[::-1])
    bc = np.zeros((3, 3, 2), np.int8)
    if per is not None:
        bc[:, per, :] = W.BC_P
    N = [n[J] + (J != per) for J in range(3)]
    at = rng.permutation(N[0] * N[1] * N[2])[:3 * size].reshape(3, size)
    sup = np.stack([at % N[0], at // N[0] % N[1], at // (N[0] * N[1])], -1)
    avg = [W.Average(sup, np.array([0, 1, 2], np.int8), np.array([0.01, -0.02, 0.015]), set_id=0)]
    o = OSolver(n, lam, mu, bc, (), avg, r0_factor=1.3, finite_strain=fs)
    g = F.Solver(n, lam, mu, bc, (), avg, r0_factor=1.3, precision="fp64", finite_strain=fs)
    u = rng.standard_normal(o.zeros().shape) * 2e-2
    parts = o.iterate_parts(u)
    p, pt, sums = g.stage_residual(u)
    assert np.abs(pt - parts["ptil"]).max() <= 1e-12 * np.abs(parts["ptil"]).max()
    assert np.abs(p - parts["p"]).max() <= 1e-12 * np.abs(parts["p"]).max()
    assert abs(sums[0] - parts["pnorm2"]) <= 1e-11 * parts["pnorm2"]


@pytest.mark.parametrize("n", [(30, 6, 3), (32, 7, 2), (60, 2, 9), (63, 13, 33)])
@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("fs", [False, True])
def test_march_with_singular_modes(n, f64, fs):
    """The instance for an obstacle or singular modes (here: no fixed face), whose passes with FP32
    and with FP64 stresses are one launch: one step from random fields as above."""
    F = _lib()
    print(f"[march] n={n} free faces fp64_stress={f64} finite_strain={fs}", flush=True)
    rng = np.random.default_rng(1800 + n[0])
    lam = rng.uniform(0.4, 2.5, n[::-1]); mu = rng.uniform(0.3, 1.8, n[::-1])
    bc = np.zeros((3, 3, 2), np.int8)
    o = OSolver(n, lam, mu, bc, r0_factor=1.3, finite_strain=fs)
    g = F.Solver(n, lam, mu, bc, r0_factor=1.3, precision="fp32", finite_strain=fs)
    u, delta, e, p_prev, R_prev = (rng.standard_normal(o.zeros().shape) * sc for sc in (2e-2, 1e-3, 2e-2, 2e-2, 2e-2))
    pe = o.iterate_parts(u)["p"]
    k0d = -o.reference_term(tetra2.tet_gradients(delta, o.plan))
    p, R, dR, dY, sums = g.stage_residual_form(u, delta, e, p_prev, R_prev, 3, fp64_stress=int(f64))
    tol = 2e-6 if f64 else 2e-5
    assert np.abs(p - pe).max() <= tol * np.abs(pe).max()
    assert abs(sums[0] - np.sum(pe ** 2)) <= 10 * tol * np.sum(pe ** 2)
    Re = pe + k0d - e
    assert np.abs(R - Re).max() <= tol * np.abs(Re).max()
    dYe = pe - p_prev + k0d
    assert np.abs(dY - dYe).max() <= tol * np.abs(dYe).max()


@pytest.mark.parametrize("e", [0, 80])
@pytest.mark.parametrize("n", [(6, 5, 4), (40, 9, 7)])
def test_fp32_literal_stress_norm_is_summed_in_fp64(n, e):
    """The literal residual pass on FP32 fields: uniaxial strain whose stress, 2 mu a = 2049 2051 2^(e - 32), is an
    FP32 number but its square is not (and for e = 80 exceeds FP32).  Its sum over the voxels is exact in
    FP64 up to its additions, at most as many as voxels."""
    F = _lib()
    lam = np.zeros(n[::-1]); mu = np.full(n[::-1], 2049.0 * 2.0 ** (e - 11))
    g = F.Solver(n, lam, mu, np.zeros((3, 3, 2), np.int8), precision="fp32", acv="U")
    u = np.zeros((3, n[2] + 1, n[1] + 1, n[0] + 1))
    u[0] = np.arange(n[0] + 1) * (2051.0 * 2.0 ** -22)
    print(f"[march] literal FP32 stress norm n={n} e={e}", flush=True)
    _, _, sums = g.stage_residual(u)
    exact = lam.size * (2049.0 * 2051.0 * 2.0 ** (e - 32)) ** 2
    assert abs(sums[1] - exact) <= lam.size * 2.0 ** -53 * exact
