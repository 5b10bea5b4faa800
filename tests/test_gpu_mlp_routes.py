"""Network steps and predictions on both sides of the lines between the block kernel and
layer-by-layer launches, against the FP64 oracle (1e-5 on predictions and loss, 1e-4 on
each gradient tensor); and few samples of a wide network, which leave the block kernel
to few workgroups, are no slower than layer by layer."""
import numpy as np
import pytest
import torch

from oracle import mlp as O
from paper_1305_1183_amd import kf
from test_gpu_mlp import rel, setup

pytestmark = pytest.mark.gpu

# (d, h, layers, n): block kernel of the general and the tiled widths at their edges
SHAPES = [(480, 480, 2, 4099), (5, 200, 2, 4097), (33, 300, 3, 4111), (40, 200, 5, 16390), (8, 129, 1, 4095),
          (129, 31, 2, 50), (128, 16, 2, 4100), (7, 63, 2, 4098), (160, 32, 2, 4100), (64, 32, 3, 4100), (480, 64, 2, 70)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_step_matches_oracle(shape):
    d, h, L, n = shape
    m, p, X, y, P, Xd, yd, ws, wsb = setup(d, h, L, n, 12)
    G = torch.full_like(P, float("nan"))
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    pred = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
    kf.kf_mlp_forward(m, P.data_ptr(), Xd.data_ptr(), n, pred.data_ptr(), ws.data_ptr(), wsb)
    kf.kf_mlp_loss_grad(m, P.data_ptr(), Xd.data_ptr(), yd.data_ptr(), n, G.data_ptr(), loss.data_ptr(), ws.data_ptr(), wsb)
    torch.cuda.synchronize()
    ref, _ = O.forward(p, X, d, h, L)
    assert rel(pred.cpu().numpy(), ref) <= 1e-5
    lref, gref = O.loss_grad(p, X, y, d, h, L)
    assert abs(loss.item() - lref) <= 1e-5 * abs(lref)
    g = G.cpu().numpy()
    for (w, b, i, o) in O.layout(d, h, L)[0]:
        assert rel(g[w:w + i * o], gref[w:w + i * o]) <= 1e-4, ("W", w)
        assert rel(g[b:b + o], gref[b:b + o]) <= 1e-4, ("b", b)


@pytest.mark.parametrize("shape", [(480, 480, 8, 16), (480, 400, 3, 64)], ids=str)
def test_wide_networks_of_few_samples_are_not_slower(shape):
    """2 d h + ... products of 16 samples: layer by layer 1.1 ms for 16 layers of 480; the
    block kernel took four times that. Bound: twice a launch a layer at 20 us."""
    d, h, L, n = shape
    m, p, X, y, P, Xd, yd, ws, wsb = setup(d, h, L, n, 3)
    G, loss = torch.empty_like(P), torch.zeros(1, device="cuda")

    def step():
        kf.kf_mlp_loss_grad(m, P.data_ptr(), Xd.data_ptr(), yd.data_ptr(), n, G.data_ptr(), loss.data_ptr(), ws.data_ptr(), wsb)
    for _ in range(5):
        step()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(20):
        step()
    b.record()
    torch.cuda.synchronize()
    us = a.elapsed_time(b) / 20 * 1e3
    assert us <= 2 * 20 * (3 * L + 3), us
