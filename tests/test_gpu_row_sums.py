"""Row sums in the library's geometry end every 256 columns of FP32 and are merged as
pairs, as in small workgroups of one float4 a lane: the same bits, whether a wave
streams the rows or a strip is wider, at ragged and at long rows."""
import numpy as np
import pytest

import seqcheck as SC
from paper_1305_1183_amd import workloads as WL

pytestmark = pytest.mark.gpu

SHAPES = [(1030, 5003), (2600, 2500), (700, 9001), (3001, 2304), (20003, 301), (90001, 70), (40, 200003), (512, 16384),
          (6000, 1025)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("name,out", [("bicgk", "q"), ("gesummv", "y")])
def test_same_bits_as_small_workgroups(name, out, shape):
    m, n = shape
    print("case row sums", name, m, n, flush=True)
    arrays, scal = WL.make(name, m, n, seed=71)
    _, prog, host = SC.run_gpu(name, m, n, arrays, scal)
    _, _, small = SC.run_gpu(name, m, n, arrays, scal, mat_k=1, mat_waves=4, mat_group=4)
    SC.check_against_oracle(name, m, n, host, SC.oracle_outputs(name, arrays, scal, n))
    assert np.array_equal(host[out].view(np.uint32), small[out].view(np.uint32))
    k = prog.describe()["kernels"][0]["params"]
    assert (k["strips"] if k.get("schedule") == "row-stream" else k["row_sums"]) == -(-n // 256)
