"""The network's line kernels at the edges of their tiles: lines of one node more or less than
the 16- and 32-node pieces, grids of one chunk and of many, short last chunks, every split of
the modes over the MFMA slots (m = 1 .. 6), and networks of no, one and two blocks.

Against the FP64 oracle: outputs to 1e-2 relative (BF16's unit roundoff 2^-9 over a handful of
roundings per layer, as in test_gpu_nn.py), gradients to 2e-2 (twice the layers: the way there
and the way back)."""
import numpy as np
import pytest

from oracle import nn as onn
from test_gpu_nn import _cos, _feat_dev, _net_case, _rel, _torch

pytestmark = pytest.mark.gpu

CASES = [((2, 3, 2), 2, 1), ((15, 4, 5), 3, 1), ((16, 5, 3), 5, 2), ((17, 9, 2), 4, 1), ((31, 7, 4), 6, 2),
         ((32, 6, 3), 1, 2), ((33, 17, 5), 6, 1), ((48, 5, 17), 2, 2), ((257, 3, 2), 6, 1), ((5, 103, 101), 6, 2),
         ((33, 5, 3), 6, 0)]


@pytest.mark.parametrize("N,modes,blocks", CASES)
def test_tile_edges_match_oracle(N, modes, blocks):
    torch, F = _torch()
    print(f"[nn tiles] N={N} m={modes} B={blocks}", flush=True)
    shape, vec, f, t = _net_case(21, N, modes, blocks)
    fd, fval = _feat_dev(torch, f)
    p = onn.unflatten(vec, **shape)
    y, cache = onn.forward(p, fval, N, blocks=blocks, m=modes)
    net = F.Net(modes, blocks)
    net.set_params(vec)
    net.bind(N, training=False)
    assert _rel(net.forward(fd).cpu().numpy().astype(np.float64), y) <= 1e-2
    L, dy = onn.loss(y, t, fval[:, 9:12])
    gr = onn.flatten(onn.backward(p, cache, dy), **shape)
    net.bind(N, training=True)
    net.train_step(fd, torch.as_tensor(np.ascontiguousarray(t.T, np.float32), device="cuda"))
    g = net.grad().cpu().numpy().astype(np.float64)
    assert _cos(g, gr) >= 0.999 and _rel(g, gr) <= 2e-2, (_cos(g, gr), _rel(g, gr))
    # inference on the training workspace gives the same values
    assert _rel(net.forward(fd).cpu().numpy().astype(np.float64), y) <= 1e-2
