"""The network step at the edges of its 16 x 16 tiles and on both of its routes
(blocks of 16 samples through all layers; layer by layer for wide networks and
smaller workspaces), against the FP64 oracle. Tolerances as for the other
network tests: 1e-5 on predictions and loss, 1e-4 on each gradient tensor."""
import numpy as np
import pytest
import torch

from oracle import mlp as O
from paper_1305_1183_amd import kf
from test_gpu_mlp import rel, setup

pytestmark = pytest.mark.gpu

# (d, h, layers, n): single entries, one below / at / above a tile, the widest block and the first width past it
SHAPES = [(1, 1, 1, 1), (3, 15, 2, 15), (16, 16, 1, 16), (17, 17, 4, 17), (33, 65, 3, 63), (32, 128, 3, 65),
          (5, 200, 2, 300), (64, 64, 1, 16), (96, 32, 5, 40), (160, 128, 2, 31), (480, 480, 1, 19), (32, 481, 2, 33), (481, 16, 2, 33)]


def least_floats(h, L, n):
    """Workspace of the layer-by-layer route: L activation and two gradient buffers, prediction and its gradient."""
    return (L + 2) * n * h + 2 * n + 64


@pytest.mark.parametrize("small", [False, True], ids=["workspace", "least-workspace"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_step_matches_oracle(shape, small):
    d, h, L, n = shape
    m, p, X, y, P, Xd, yd, ws, wsb = setup(d, h, L, n, 12)
    if small:
        wsb = 4 * least_floats(h, L, n)
    G = torch.full_like(P, float("nan"))
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    pred = torch.empty(n, dtype=torch.float32, device="cuda")
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


def test_smaller_workspace_is_still_refused_below_the_least():
    m, p, X, y, P, Xd, yd, ws, wsb = setup(32, 64, 3, 20, 1)
    G, out = torch.empty_like(P), torch.empty(20, device="cuda")
    wsb = 4 * least_floats(64, 3, 20) - 4
    with pytest.raises(kf.KFError):
        kf.kf_mlp_loss_grad(m, P.data_ptr(), Xd.data_ptr(), yd.data_ptr(), 20, G.data_ptr(), 0, ws.data_ptr(), wsb)
    with pytest.raises(kf.KFError):
        kf.kf_mlp_forward(m, P.data_ptr(), Xd.data_ptr(), 20, out.data_ptr(), ws.data_ptr(), wsb)
