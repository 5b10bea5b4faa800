"""Finishing launches of column and row partials against the FP64 oracle (1e-5 log2 n):
column counts around a workgroup's 64 columns, row counts from one block to more blocks
than lane groups that share them, and more column strips than partials loaded at once;
integer inputs, whose sums FP32 holds, come out exactly."""
import numpy as np
import pytest

import seqcheck as SC
from paper_1305_1183_amd import workloads as WL

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (70, 63), (300, 64), (33, 65), (4099, 127), (257, 1021), (9000, 60), (20011, 130), (515, 9001)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("name", ["bicgk", "atax", "gemver"])
def test_finished_sums(name, shape):
    m, n = shape
    print("case finish", name, m, n, flush=True)
    arrays, scal = WL.make(name, m, n, seed=61)
    _, _, host = SC.run_gpu(name, m, n, arrays, scal)
    SC.check_against_oracle(name, m, n, host, SC.oracle_outputs(name, arrays, scal, n))


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_integer_sums_are_exact(shape):
    m, n = shape
    rng = np.random.default_rng(m * 31 + n)
    ld = (n + 3) // 4 * 4
    A = np.zeros((m, ld), np.float32)
    A[:, :n] = rng.integers(-3, 4, (m, n))
    p, r = rng.integers(-3, 4, n).astype(np.float32), rng.integers(-3, 4, m).astype(np.float32)
    print("case finish exact", m, n, flush=True)
    _, _, host = SC.run_gpu("bicgk", m, n, {"A": A, "p": p, "r": r}, {})
    np.testing.assert_array_equal(host["q"], (A[:, :n].astype(np.float64) @ p).astype(np.float32))
    np.testing.assert_array_equal(host["s"], (A[:, :n].T.astype(np.float64) @ r).astype(np.float32))
