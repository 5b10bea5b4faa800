"""Row-resident kernels on narrow rows, where eight teams of one wave walk rows of
their own: one, two, four and eight float4 per lane, ragged columns, fewer rows than
teams, partial row groups, and every kernel shape that feeds a gemv into a gemtv
(plain, with stored rank-1 updates, with a y0), against the FP64 oracle within the
suite's tolerance 1e-5 log2 n."""
import json

import pytest

import seqcheck as SC
from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S
from paper_1305_1183_amd import workloads as WL

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (3, 5), (7, 255), (33, 256), (31, 257), (129, 511), (64, 1024), (257, 1023), (1000, 1025), (515, 2047),
          (70, 2048), (40, 2049)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_single_pass_atax(shape):
    m, n = shape
    arrays, scal = WL.make("atax", m, n, seed=31)
    _, prog, host = SC.run_gpu("atax", m, n, arrays, scal)
    SC.check_against_oracle("atax", m, n, host, SC.oracle_outputs("atax", arrays, scal, n))
    (k,) = prog.describe()["kernels"]
    assert k["params"]["teams"] == (8 if n <= 2048 else 1)


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("name", ["bicgk", "gesummv", "gemver", "sgemvt"])
def test_every_sequence_on_the_schedule(name, shape):
    m, n = shape
    arrays, scal = WL.make(name, m, n, seed=32)
    _, prog, host = SC.run_gpu(name, m, n, arrays, scal, mat_sched=1)
    SC.check_against_oracle(name, m, n, host, SC.oracle_outputs(name, arrays, scal, n))


@pytest.mark.parametrize("n", [1, 5, 256, 600, 1023, 2048])
@pytest.mark.parametrize("name", ["sgemvt", "gemver"])
def test_column_major_single_pass(name, n):
    """gemv feeds gemtv on the storage of A^T (and GEMVER stores B in the same pass)."""
    import numpy as np
    import torch
    m, cols = n, 90                              # storage: 90 rows of n
    arrays, scal = WL.make(name, m, cols, seed=33)
    ref = SC.oracle_outputs(name, arrays, scal, cols)
    q = S.by_name(name, m, cols, scal, layout=kf.KF_COL_MAJOR)
    ld = q.shapes["A"][1]
    At = np.full((cols, ld), np.nan, np.float32)
    At[:, :m] = arrays["A"][:, :cols].T
    dev = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in dict(arrays, A=At).items()}
    prog = q.compile("fused").bind(**dev)
    assert prog.num_kernels == 1 and json.loads(kf.kf_plan_describe(prog.plan))["kernels"][0]["params"]["teams"] in (1, 8)
    out = {k: v.cpu().numpy() for k, v in prog.run().items()}
    if "B" in out:
        out["B"] = np.ascontiguousarray(out["B"][:, :m].T)
        ref["B"] = ref["B"][:, :cols]
    for k, r in ref.items():
        assert WL.rel_l2(out[k], r) <= WL.tolerance(name, m, cols), k
