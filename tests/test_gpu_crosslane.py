"""Cross-lane reductions: row sums of every group size and merges of every wave
count on small integers, whose sums are exact in FP32 in any order, so one wrong
lane pairing shows as a wrong integer (tolerance 0)."""
import numpy as np
import pytest

from paper_1305_1183_amd import inputs as I
from seqcheck import run_gpu

pytestmark = pytest.mark.gpu

M, N = 70, 519


def operands():
    # |sum| <= 519 * 8 * 8 < 2^24
    return {"A": np.ascontiguousarray(np.pad(I.small_ints(11, 0, M * N, -8, 8).reshape(M, N), ((0, 0), (0, 1)))),
            "p": I.small_ints(11, 1, N, -8, 8), "r": I.small_ints(11, 2, M, -8, 8)}


STRIP = [dict(mat_k=1, mat_waves=w, mat_group=g, mat_rows=w * g * 2) for g in (1, 2, 4, 8, 16) for w in (1, 4)]
ROWS = [dict(mat_sched=1, mat_waves=w, mat_group=g, mat_rows=2 * g)
        for w, g in ((1, 1), (1, 16), (2, 2), (4, 8), (8, 4), (8, 8), (16, 1), (16, 2), (16, 4))]


@pytest.mark.parametrize("params", STRIP + ROWS, ids=lambda p: "-".join(str(v) for v in p.values()))
def test_row_and_column_sums_of_integers(params):
    a = operands()
    _, _, host = run_gpu("bicgk", M, N, a, {}, **params)
    A = a["A"][:, :N]
    assert np.array_equal(host["q"], (A.astype(np.float64) @ a["p"]).astype(np.float32))
    assert np.array_equal(host["s"], (A.astype(np.float64).T @ a["r"]).astype(np.float32))
