"""BF16 and FP8 matrices read in requested units of four elements: large ones keep 24
waves a CU with two rows a step, as a unit carries a half or a quarter of the bytes."""
import json

import pytest

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S


@pytest.mark.parametrize("fmt", ["bf16", "fp8"])
@pytest.mark.parametrize("n,large", [(5003, False), (8192, True), (16384, True), (32768, True)])
def test_waves(fmt, n, large):
    q = S.bicgk_q(n, n, fmt)
    p = kf.kf_compile(q.script, mode="fused", flags=kf.KF_COMPILE_CODEGEN_ONLY, mat_unit=4)
    k = json.loads(kf.kf_plan_describe(p))["kernels"][0]
    kf.kf_plan_destroy(p)
    assert (k["params"]["waves"], k["params"]["group"]) == ((8, 2) if large else (16, 1))
    if large:
        assert k["launches"][0]["grid"] * k["launches"][0]["block"] >= 256 * 20 * 64
