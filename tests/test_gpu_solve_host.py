"""What a solve shares with its process: the pinned words through which it reports, other threads'
captures and solves."""
import threading

import numpy as np
import pytest

import workloads as W
from test_gpu_parity import _lib

pytestmark = pytest.mark.gpu


def _solver(F, n, seed=1, precision="fp32", **kw):
    """A heterogeneous block on its fixed bottom, the middle of its top moved."""
    rng = np.random.default_rng(seed)
    lam = rng.uniform(0.5, 3.0, n[::-1]); mu = rng.uniform(0.5, 2.0, n[::-1])
    bc = np.zeros((3, 3, 2), np.int8)
    bc[:, 2, 0] = 1
    top = W.Strong(np.array([[n[0] // 2, n[1] // 2, n[2]]]), np.array([2], np.int8), np.array([1e-2]))
    return F.Solver(n, lam, mu, bc, strong=[top], precision=precision, tol=0.0, **kw)


def test_solve_beside_another_threads_capture():
    """The first solve of a handle, and the end of handles, leave a graph alone that another thread is
    capturing meanwhile (in torch's default mode, in which allocations of any thread are refused)."""
    F = _lib()
    import torch
    n = (24, 24, 24)
    ref, g = _solver(F, n, max_iter=20), _solver(F, n, max_iter=20)
    ref.solve()
    # 64 slots a slab: the last handle's slot is in a slab of its own, which goes with it
    many = [_solver(F, (4, 4, 4), max_iter=1) for _ in range(66)]
    for s in many:
        s.solve()
    torch.cuda.synchronize()
    x = torch.ones(1000, device="cuda")
    y = torch.zeros_like(x)
    begun, over, rcs = threading.Event(), threading.Event(), []

    def work():
        begun.wait()
        try:
            rcs.append(F.load().fftc_solve(g.h, g.u.data_ptr(), 1, None))
            for s in many:
                F.fftc_destroy(s.h)
                s.h = None
        finally:
            over.set()

    th = threading.Thread(target=work)
    th.start()
    graph = torch.cuda.CUDAGraph()
    stream = torch.cuda.Stream()
    print("[solve host] solve and destroy beside a capture", flush=True)
    with torch.cuda.graph(graph, stream=stream):
        y.add_(x)
        begun.set()
        assert over.wait(60)
        y.add_(x)
    th.join()
    assert rcs == [F.FFTC_E_NOCONV] and torch.equal(g.u, ref.u)
    for k in range(1, 4):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, torch.full_like(y, 2.0 * k))
