"""Every launch of a plan has fewer than 2^32 threads, the most HIP takes, also for the
tallest matrices that the card holds, whatever schedule the library picks."""
import json

import pytest

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S


@pytest.mark.parametrize("mode", ["fused", "unfused"])
@pytest.mark.parametrize("seq", ["bicgk", "gesummv", "gemver", "sgemvt", "atax", "bicgk_fp8", "gemver_bf16"])
def test_threads_per_launch(seq, mode):
    for m, n in ((1 << 26, 300), ((1 << 26) + 5, 257), (70_000_000, 512), (240_000_000, 64), (240_000_000, 200), (1 << 28, 4)):
        if "_" in seq:
            name, fmt = seq.split("_")
            q = S.bicgk_q(m, n, fmt) if name == "bicgk" else S.gemver_q(m, n, 1.5, 0.75, fmt)
        else:
            q = S.by_name(seq, m, n, {"alpha": 1.5, "beta": 0.75})
        p = kf.kf_compile(q.script, mode=mode, flags=kf.KF_COMPILE_CODEGEN_ONLY)
        for k in json.loads(kf.kf_plan_describe(p))["kernels"]:
            for l in k["launches"]:
                assert 0 < l["grid"] * l["block"] < 1 << 32, (seq, m, n, k["params"], l)
        kf.kf_plan_destroy(p)
