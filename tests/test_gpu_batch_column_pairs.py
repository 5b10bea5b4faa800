"""Batched GEMVER above n = 512, where a lane has every row of a block: terms 2^24, 1 and
-2^24 of a column in rows that different steps take (and that four row groups would
hold apart) leave the 1 in x, which plain FP32 addition of the steps rounds away."""
import numpy as np
import pytest
import torch

from paper_1305_1183_amd import batched as B
from paper_1305_1183_amd import kf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [513, 700, 1024, 1500, 2047])
def test_cancelling_steps(n):
    print("case batched column pairs", n, flush=True)
    bt = B.Batch(np.array([B.GEMVER], np.int32), np.array([n]), np.ones(1, np.float32), np.ones(1, np.float32),
                 kf.batch_opts())
    host = np.zeros(bt.elems, np.float32)
    off, ld = bt.offset(0, "A")
    A = host[off:off + n * ld].reshape(n, ld)
    want = np.zeros(n)
    rng = np.random.default_rng(n)
    for j in range(n):
        start = int(rng.integers(0, max(1, n // 64))) * 64 % (n - 20)
        start -= start % 64                               # inside one row block, whatever its rows
        a, b, c = rng.permutation([0, 9, 18])
        A[start + a, j], A[start + b, j], A[start + c, j] = 2.0 ** 24, 1.0, -2.0 ** 24
        want[j] = 1.0
    o, _ = bt.offset(0, "y")
    host[o:o + n] = 1.0
    bt.upload(host)
    for _ in range(2):
        bt.run(0)
    torch.cuda.synchronize()
    assert bt.error() == 0
    got = bt.outputs(bt.arena.cpu().numpy(), 0)
    assert np.array_equal(got["x"], want.astype(np.float32))
