"""A batch whose instances all take the default tiles runs in a kernel without the rest
of the tile menu; one that asks for another tile runs in the kernel with the whole menu.
Instances that take the same tile in both get the same bits."""
import numpy as np
import pytest
import torch

from paper_1305_1183_amd import batched as B
from paper_1305_1183_amd import kf

pytestmark = pytest.mark.gpu

NS = [1, 33, 64, 65, 128, 129, 256, 300, 512, 513, 1024, 1025, 2048]


@pytest.mark.parametrize("which", [0, 1])
@pytest.mark.parametrize("kind", [B.BICGK, B.GEMVER])
def test_default_tiles_in_both_kernels(kind, which):
    ns = np.array(NS)
    kinds = np.full(len(ns), kind, np.int32)
    sc = np.full(len(ns), 1.25, np.float32)
    out = []
    for other in (0, 1):
        bt = B.Batch(kinds, ns, sc, sc, kf.batch_opts(tiles={kind: [0, 0, 0, other, 0, 0]}))
        print("case batch menu", kind, which, other, flush=True)
        bt.upload(bt.host_arena(seed=4))
        for _ in range(2):
            bt.run(which)
        torch.cuda.synchronize()
        assert bt.error() == 0
        host = bt.arena.cpu().numpy()
        out.append([bt.outputs(host, i) for i in range(len(ns))])
    for i, n in enumerate(NS):
        if not 256 < n <= 512:
            for name, v in out[0][i].items():
                assert np.array_equal(np.nan_to_num(v), np.nan_to_num(out[1][i][name])), (n, name)
