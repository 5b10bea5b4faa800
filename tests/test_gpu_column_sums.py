"""Column sums of strip kernels in the library's geometry, in each way a wave adds its
rows (row by row, the sum of a step, pairs) and with several row blocks per workgroup,
on ragged rows and columns: small integers, whose sums FP32 holds exactly in any order,
so one row dropped, doubled or taken from another block shows as a wrong integer."""
import pytest
import torch

from paper_1305_1183_amd import sequences as S

pytestmark = pytest.mark.gpu

# (sequence, storage, rows, cols, how, several blocks per workgroup)
CASES = [("bicgk", "f32", 2447, 2441, "pairs", False), ("bicgk", "f32", 20011, 701, "steps", False),
         ("bicgk", "f32", 301, 66003, "steps", False), ("bicgk", "f32", 5003, 5001, "rows", False),
         ("bicgk", "f32", 18001, 33003, "rows", True), ("bicgk", "f32", 17009, 16390, "steps", False),
         ("bicgk", "bf16", 8193, 4099, "steps", False), ("bicgk", "bf16", 4095, 4090, "steps", True),
         ("bicgk", "fp8", 8209, 8191, "steps", False), ("bicgk", "fp8", 9001, 1500, "steps", True),
         ("bicgk", "fp8", 40009, 33, "pairs", False), ("gemver", "f32", 2500, 2491, "pairs", False),
         ("gemver", "f32", 9001, 9001, "pairs", False), ("gemver", "f32", 4099, 4096, "pairs", False),
         ("gemver", "f32", 26001, 19999, "pairs", True)]


def ints(g, lo, hi, *shape):
    return torch.randint(lo, hi + 1, shape, generator=g, device="cuda").float()


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v) for v in c))
def test_integer_sums(case):
    seq, fmt, m, n, how, several = case
    print("case column sums", case, flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + n)
    if fmt == "f32":
        q = S.by_name(seq, m, n, {"alpha": 1.0, "beta": 1.0})
        A = ints(g, -3, 3, *q.shapes["A"])
        A[:, n:] = float("nan")
        dev = {"A": A}
    else:
        q = S.bicgk_q(m, n, fmt)
        A = ints(g, -3, 3, *q.shapes["A"])
        A[:, n:] = float("nan")
        codes = A.to(torch.bfloat16).view(torch.int16) if fmt == "bf16" else A.to(torch.float8_e4m3fn).view(torch.uint8)
        dev = {"A": codes, "A_scale": torch.ones(m, device="cuda")}
    rowv, colv = (["r"], ["p"]) if seq == "bicgk" else (["u1", "u2", "y"], ["v1", "v2", "z"])
    dev.update({k: ints(g, -3, 3, m) for k in rowv}, **{k: ints(g, -3, 3, n) for k in colv})
    prog = q.compile("fused").bind(**dev)
    k = prog.describe()["kernels"][0]["params"]
    assert k["column_sums"] == how and (k["turns"] > 1) == several, k
    for _ in range(2):
        out = prog.run()
    torch.cuda.synchronize()
    B = A[:, :n].double()
    if seq == "bicgk":
        assert torch.equal(out["s"].double(), B.t() @ dev["r"].double())
        assert torch.equal(out["q"].double(), B @ dev["p"].double())
    else:
        for u, v in (("u1", "v1"), ("u2", "v2")):
            B.addr_(dev[u].double(), dev[v].double())
        assert torch.equal(out["B"][:, :n].double(), B)
        x = B.t() @ dev["y"].double() + dev["z"].double()
        assert torch.equal(out["x"].double(), x)
