"""Column sums of single-wave teams reach the finishing launch unrounded where a matrix
has few rows: 2^24 + 1 of one workgroup and 1 of another add up to 2^24 + 2, which an
FP32 total of the first workgroup loses (exact, tolerance 0)."""
import pytest
import torch

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [64, 100, 700, 1024])
@pytest.mark.parametrize("n", [1, 300, 513, 1026, 2048])
@pytest.mark.parametrize("name", ["atax", "sgemvt"])
def test_total_of_a_workgroup(name, m, n):
    print("case", name, m, n, flush=True)
    col = name == "sgemvt"
    layout = kf.KF_COL_MAJOR if col else kf.KF_ROW_MAJOR
    q = S.by_name(name, *((n, m) if col else (m, n)), {"alpha": 1.0, "beta": 1.0}, layout=layout)
    prog = q.compile(mode="fused")
    k = prog.describe()["kernels"][0]
    assert k["params"]["teams"] == 8 and k["params"]["row_blocks"] > 1
    dev = {v: torch.zeros(q.shapes[v], device="cuda") for v in q.inputs}
    # rows 0 and 4 belong to different teams of the first workgroup, the last row to another one
    for row, v in ((0, 4096.0), (4, 1.0), (m - 1, 1.0)):
        dev["A"][row, 0] = v
    if col:
        # x = A^T y in storage rows, w = A x in storage columns: w[0] = sum of a^2
        dev["y"][0] = 1.0
    else:
        dev["x"][0] = 1.0
    out = prog.bind(**dev).run()
    got = out["w" if col else "y"].cpu()
    want = torch.zeros(n)
    want[0] = 2.0 ** 24 + 2
    assert torch.equal(got, want)
