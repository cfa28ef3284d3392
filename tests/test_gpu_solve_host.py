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


@pytest.mark.parametrize("shared", [False, True])
def test_solves_from_two_threads(shared):
    """Two handles solved over and over from two threads, on a stream each or on one: every solve is
    bitwise the handle's solve alone."""
    F = _lib()
    import torch
    streams = [torch.cuda.Stream() for _ in range(2)]
    if shared:
        streams[1] = streams[0]
    hs = []
    for k, (n, prec) in enumerate([((20, 16, 18), "fp64"), ((48, 40, 32), "fp32")]):
        with torch.cuda.stream(streams[k]):
            hs.append(_solver(F, n, seed=3 + k, precision=prec, max_iter=60))
    ref = []
    for g in hs:
        g.solve()
        ref.append(g.u.clone())
    torch.cuda.synchronize()
    print(f"[solve host] two threads, shared stream {shared}", flush=True)
    bad = []

    def work(k):
        torch.cuda.set_device(0)
        for _ in range(8):
            rep = F.fftc_report()
            rc = F.load().fftc_solve(hs[k].h, hs[k].u.data_ptr(), 1, rep)
            if rc != F.FFTC_E_NOCONV or rep.iterations != 60 or not torch.equal(hs[k].u, ref[k]):
                bad.append((k, rc, rep.iterations))

    ths = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ths:
        t.start()
    for t in ths:
        t.join()
    assert not bad


def test_slots_of_two_slabs_report_their_own_solves():
    """80 handles kept alive over two slabs of slots: each solve ends at its own iteration with its own
    result, and so do new handles in the slots that others gave back."""
    F = _lib()
    import torch
    want = {}

    def check(k):
        it = 1 + k % 7
        g = _solver(F, (6, 5, 4), max_iter=it)
        rc, rep = g.solve()
        assert rc == F.FFTC_E_NOCONV and rep.iterations == it, (k, rc, rep.iterations)
        assert torch.equal(g.u, want.setdefault(it, g.u.clone()))
        return g

    print("[solve host] 80 handles", flush=True)
    hs = [check(k) for k in range(80)]
    assert len({float(u.abs().sum()) for u in want.values()}) == 7
    for k in list(range(79, 62, -1)) + list(range(0, 60, 3)):
        F.fftc_destroy(hs[k].h)
        hs[k].h = None
    hs += [check(k) for k in range(30)]
