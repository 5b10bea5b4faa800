"""Batched GEMVER cut into row blocks: blocks that end inside a step, whose B other
workgroups read, keep the padding of B as it was and an infinite entry in a block's last
row infinite (rows past a block must not enter its column sums), over several launches."""
import numpy as np
import pytest
import torch

import oracle
from paper_1305_1183_amd import batched as B
from paper_1305_1183_amd import kf
from paper_1305_1183_amd import workloads as WL

pytestmark = pytest.mark.gpu

NS = [5, 129, 131, 257, 389, 513, 777, 1025, 2047]


@pytest.mark.parametrize("which", [0, 1])
@pytest.mark.parametrize("steps", [1, 3, 0])
def test_split_gemver_blocks(steps, which):
    rows = {1: [steps * r for r in kf.BATCH_ROWS_PER_STEP]}     # 0: the default rows per block
    ns = np.array(NS)
    bt = B.Batch(np.ones(len(ns), np.int32), ns, np.full(len(ns), 1.25, np.float32), np.full(len(ns), 0.75, np.float32),
                 kf.batch_opts(rows=rows))
    host = bt.host_arena(seed=3)
    col = {}
    for i, n in enumerate(NS):
        off, ld = bt.offset(i, "A")
        A = host[off:off + n * ld].reshape(n, ld)
        A[n - 1, n // 2] = np.inf
        host[bt.offset(i, "y")[0] + n - 1] = 1.0
        off, ld = bt.offset(i, "B")
        host[off:off + n * ld] = 7.0
        col[i] = n // 2
    print("case split gemver steps=%d which=%d" % (steps, which), flush=True)
    bt.upload(host)
    for _ in range(3):
        kf.kf_batch_run(bt.h, which, bt.stream())
        torch.cuda.synchronize()
        assert bt.error() == 0
        out = bt.arena.cpu().numpy()
        for i, n in enumerate(NS):
            off, ld = bt.offset(i, "A")
            A = host[off:off + n * ld].reshape(n, ld).copy()
            A[n - 1, col[i]] = 0.0
            v = [host[bt.offset(i, k)[0]:bt.offset(i, k)[0] + n] for k in B.INPUTS[B.GEMVER]]
            Br, xr, _ = oracle.gemver(1.25, 0.75, A, *v, cols=n)
            got = bt.outputs(out, i)
            assert np.all(got["B"][:, n:] == 7.0), n
            assert np.isposinf(got["B"][n - 1, col[i]]) and np.isposinf(got["x"][col[i]]), n
            keep = np.arange(n) != col[i]
            tol = WL.tolerance("gemver", n, n)
            assert WL.rel_l2(got["x"][keep], xr[keep]) <= tol, n
            Bg = got["B"][:, :n].copy()
            Bg[n - 1, col[i]] = Br[n - 1, col[i]]
            assert WL.rel_l2(Bg, Br) <= tol, n
        bt.arena.copy_(torch.from_numpy(host).cuda())
