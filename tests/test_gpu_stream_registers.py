"""Row-stream kernels whose operands leave registers for fewer rows a wave, against float64."""
import pytest
import torch

from test_stream_registers_host import products

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmts,group", [(("bf16",), 4), (("bf16", "f32", "f32"), 2), (("bf16",) * 2 + ("f32",) * 3, 1)])
@pytest.mark.parametrize("m,n", [(1030, 8200), (1027, 8193), (4102, 8200), (4099, 8193)])
def test_sums(fmts, group, m, n):
    print(fmts, m, n, flush=True)
    q = products(m, n, fmts)
    gen = torch.Generator().manual_seed(m + n + len(fmts))
    dev, ref, size = {}, 0.0, 0.0
    x = torch.rand(n, generator=gen) - 0.5
    dev["x"] = x.cuda()
    for i, f in enumerate(fmts):
        name = "A%d" % i
        A = torch.rand(q.shapes[name], generator=gen) - 0.5
        if f == "bf16":
            A = A.to(torch.bfloat16)
            sc = torch.rand(m, generator=gen) + 0.5
            dev[name], dev[name + "_scale"] = A.view(torch.int16).cuda(), sc.cuda()
        else:
            sc = torch.ones(m)
            dev[name] = A.cuda()
        A = A[:, :n].double() * sc.double()[:, None]
        ref = ref + A @ x.double()
        size = size + A.abs() @ x.double().abs()
    prog = q.compile(mode="fused").bind(**dev)
    k = prog.describe()["kernels"][0]["params"]
    assert k["schedule"] == "row-stream"
    if m >= 4096:   # enough waves whatever rows they share
        assert k["group"] == group
    y = prog.run()["y"].cpu().double()
    # a strip's products: chains of at most 8 in a lane and 6 butterfly steps, two more
    # roundings for scale and store and one per matrix added
    tol = (8 + 6 + 2 + len(fmts)) * 2.0 ** -24
    assert ((y - ref).abs() <= tol * size).all(), ((y - ref).abs() / size).max()
