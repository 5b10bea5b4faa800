"""Row sums exchanged through LDS, every group size, on small integers whose sums are
exact in FP32 in any order (tolerance 0)."""
import pytest
import torch

from paper_1305_1183_amd import sequences as S

pytestmark = pytest.mark.gpu

M, N = 14147, 14203
POINTS = [{}] + [dict(mat_k=k, mat_waves=4, mat_group=g, mat_rows=64 * g) for k, g in ((1, 1), (2, 2), (1, 4), (1, 8), (1, 16))]


def test_sums_of_integers():
    gen = torch.Generator(device="cuda").manual_seed(9)
    q = S.by_name("bicgk", M, N, {})
    # |sum| <= 14203 * 8 * 8 < 2^24
    dev = {k: torch.randint(-8, 9, q.shapes[k], generator=gen, device="cuda").float() for k in q.inputs}
    A = dev["A"][:, :N].double()
    want_q, want_s = A @ dev["p"].double(), A.T.contiguous() @ dev["r"].double()
    for point in POINTS:
        print("case", point, flush=True)
        prog = q.compile(mode="fused", **point).bind(**dev)
        out = prog.run()
        assert torch.equal(out["q"].double(), want_q), point
        assert torch.equal(out["s"].double(), want_s), point
