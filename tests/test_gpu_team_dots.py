"""Row dots of one-wave teams (row-resident kernels, rows of at most 2048 columns) end
every 256 columns and meet as pairs: partial sums of 2^24, 1 and -2^24 in different
256-column parts keep the 1 that plain FP32 addition rounds away, and the bits are those
of waves that share the row (256 columns each)."""
import numpy as np
import pytest

import seqcheck as SC
from paper_1305_1183_amd import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [600, 1021, 1500, 2047])
def test_cancelling_parts(n):
    m = 40
    parts = -(-n // 256)
    A = np.zeros((m, (n + 3) // 4 * 4), np.float32)
    for i in range(m):
        a, b, c = np.random.default_rng(i).permutation(parts)[:3]
        A[i, 256 * a + 7], A[i, 256 * b + 9], A[i, 256 * c + 11] = 2.0 ** 24, 1.0, -2.0 ** 24
    x = np.ones(n, np.float32)
    _, prog, host = SC.run_gpu("atax", m, n, {"A": A, "x": x}, {})
    assert prog.describe()["kernels"][0]["params"]["teams"] == 8
    # A x is 1 in every row, and y = A^T 1 adds a few entries of each kind, all of them exact
    assert np.array_equal(host["y"], A[:, :n].sum(0, dtype=np.float64).astype(np.float32))


@pytest.mark.parametrize("shape", [(300, 700), (515, 1021), (90, 2047), (70, 256), (1000, 30)], ids=str)
def test_same_bits_as_waves_that_share_a_row(shape):
    m, n = shape
    arrays, scal = WL.make("bicgk", m, n, seed=81)
    waves = -(-n // 256)
    _, prog, team = SC.run_gpu("bicgk", m, n, arrays, scal, mat_sched=1)
    _, _, wide = SC.run_gpu("bicgk", m, n, arrays, scal, mat_sched=1, mat_waves=waves, mat_group=4, mat_rows=4)
    assert prog.describe()["kernels"][0]["params"]["teams"] == 8
    assert np.array_equal(team["q"].view(np.uint32), wide["q"].view(np.uint32))
