"""The network's line kernels with 12 to 16 x lines a workgroup (planes of more than 20,480 lines), among
them the training instance on the longest lines, which takes more than 64 KB of LDS, and a
short last chunk.  Against the network in plain FP64 PyTorch; tolerances as in test_gpu_nn_tiles.py."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import nn as onn
from test_gpu_nn import _torch

pytestmark = pytest.mark.gpu

CASES = [((33, 150, 150), 6, 2), ((20, 180, 175), 3, 2), ((257, 176, 176), 6, 1)]


def _network(torch, p, f, N, m, blocks):
    x = f @ p["Wl"].t() + p["bl"]
    cx, cy, cz = (torch.cos(math.pi * (torch.arange(v, dtype=torch.float64, device="cuda")[:, None] + 0.5)
                            * torch.arange(m, device="cuda") / v) for v in N)
    for b in range(blocks):
        h = torch.tensordot(cz.t(), x.reshape(N[2], -1), 1).reshape(m, N[1], -1)
        h = torch.einsum("yb,dyr->dbr", cy, h).reshape(m, m, N[0], 32)
        h = torch.einsum("xa,dbxc->dbac", cx, h).reshape(m ** 3, 32) / x.shape[0]
        h = torch.einsum("koc,kc->ko", p[f"Ws{b}"], h).reshape(m, m, m, 32)
        s = torch.einsum("xa,dbac->dbxc", cx, h).reshape(m, m, -1)
        s = torch.einsum("yb,dbr->dyr", cy, s).reshape(m, -1)
        x = torch.nn.functional.gelu((cz @ s).reshape(-1, 32) + x @ p[f"W{b}"].t() + p[f"c{b}"])
    h = torch.nn.functional.gelu(x @ p["Wp1"].t() + p["bp1"])
    return h @ p["Wp2"].t() + p["bp2"]


@pytest.mark.parametrize("N,modes,blocks", CASES)
def test_many_lines_a_workgroup(N, modes, blocks):
    torch, F = _torch()
    print(f"[nn lines] N={N} m={modes} B={blocks}", flush=True)
    shape = dict(width=32, modes=modes, blocks=blocks, hidden=64, cin=12, cout=3)
    vec = W.nn_init(31, [s for _, s in onn.param_layout(**shape)]).astype(np.float32)
    gen = torch.Generator(device="cuda").manual_seed(5)
    Nn = N[0] * N[1] * N[2]
    feat = torch.zeros((Nn, 16), dtype=torch.bfloat16, device="cuda")
    feat[:, :12] = torch.randn((Nn, 12), generator=gen, device="cuda").to(torch.bfloat16)
    t = torch.randn((3, Nn), generator=gen, device="cuda")
    net = F.Net(modes, blocks)
    net.set_params(vec)
    net.bind(N, training=True)
    y = net.forward(feat.view(torch.int16)).double()
    net.train_step(feat.view(torch.int16), t)
    g = net.grad().double()
    pv = torch.as_tensor(vec.astype(np.float64), device="cuda").requires_grad_(True)
    p, o = {}, 0
    for name, s in onn.param_layout(**shape):
        p[name] = pv[o:o + math.prod(s)].reshape(s)
        o += math.prod(s)
    fv, tv = feat[:, :12].double(), t.double().t()
    yr = _network(torch, p, fv, N, modes, blocks)
    loss = (yr - tv).square().sum() / (tv.square().sum() + fv[:, 9:12].square().sum())
    gr, = torch.autograd.grad(loss, pv)
    yr = yr.detach()
    assert float((y - yr).norm() / yr.norm()) <= 1e-2
    rel, cos = float((g - gr).norm() / gr.norm()), float(g @ gr / (g.norm() * gr.norm()))
    assert cos >= 0.999 and rel <= 2e-2, (cos, rel)
