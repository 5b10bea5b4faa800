"""Column sums of one to nine row blocks, which one lane or four waves finish, against float64."""
import pytest
import torch

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [31, 33, 64, 250, 256, 257, 288])
@pytest.mark.parametrize("n", [1, 3, 255, 257, 1026])
def test_bicgk(m, n):
    print("bicgk", m, n, flush=True)
    gen = torch.Generator().manual_seed(1000 * m + n)
    q = S.by_name("bicgk", m, n, {})
    host = {k: torch.rand(q.shapes[k], generator=gen) - 0.5 for k in q.inputs}
    out = q.compile(mode="fused").bind(**{k: v.cuda() for k, v in host.items()}).run()
    A, p, r = host["A"][:, :n].double(), host["p"].double(), host["r"].double()
    # s: a block's 32 rows are at most 4 a wave and 8 waves; q: 4 products a lane and 6
    # butterfly steps a strip; the rest is pairs, with a rounding each for alpha and the result
    for got, ref, size, steps in ((out["s"], A.T @ r, A.abs().T @ r.abs(), 4 + 8 + 2), (out["q"], A @ p, A.abs() @ p.abs(), 4 + 6 + 2)):
        assert ((got.cpu().double() - ref).abs() <= steps * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("m,n", [(40, 40), (159, 100), (257, 63), (70, 300)])
def test_gesummv_of_columns(m, n):
    print("gesummv", m, n, flush=True)
    gen = torch.Generator().manual_seed(1000 * m + n)
    q = S.by_name("gesummv", m, n, {"alpha": 1.5, "beta": 0.75}, layout=kf.KF_COL_MAJOR)
    host = {k: torch.rand(q.shapes[k], generator=gen) - 0.5 for k in q.inputs}
    out = q.compile(mode="fused").bind(**{k: v.cuda() for k, v in host.items()}).run()["y"].cpu().double()
    A, B, x = host["A"].double()[:, :m].T, host["B"].double()[:, :m].T, host["x"].double()
    ref, size = 1.5 * (A @ x) + 0.75 * (B @ x), 1.5 * (A.abs() @ x.abs()) + 0.75 * (B.abs() @ x.abs())
    assert ((out - ref).abs() <= (4 + 8 + 4) * 2.0 ** -24 * size).all()


def test_atax_of_few_rows():
    m, n = 40, 700
    print("atax", m, n, flush=True)
    gen = torch.Generator().manual_seed(5)
    q = S.by_name("atax", m, n, {})
    host = {k: torch.rand(q.shapes[k], generator=gen) - 0.5 for k in q.inputs}
    out = q.compile(mode="fused").bind(**{k: v.cuda() for k, v in host.items()}).run()["y"].cpu().double()
    A, x = host["A"][:, :n].double(), host["x"].double()
    size = A.abs().T @ (A.abs() @ x.abs())
    # a row's dot: 12 products a lane and 6 butterfly steps; at most all rows in one chain
    assert ((out - A.T @ (A @ x)).abs() <= (12 + 6 + 2 + m + 2) * 2.0 ** -24 * size).all()
