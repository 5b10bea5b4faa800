"""A finishing launch of few row blocks is one wave a workgroup, of more it is four."""
import json

import pytest

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S


@pytest.mark.parametrize("name,layout", [("bicgk", kf.KF_ROW_MAJOR), ("gesummv", kf.KF_COL_MAJOR), ("sgemvt", kf.KF_ROW_MAJOR)])
@pytest.mark.parametrize("m,waves", [(36, 1), (64, 1), (160, 1), (256, 1), (300, 4), (600, 4)])
def test_waves(name, layout, m, waves):
    q = S.by_name(name, m, m, {"alpha": 1.5, "beta": 0.75}, layout=layout)
    p = kf.kf_compile(q.script, mode="fused", flags=kf.KF_COMPILE_CODEGEN_ONLY)
    k = json.loads(kf.kf_plan_describe(p))["kernels"][0]
    kf.kf_plan_destroy(p)
    assert (k["params"]["row_blocks"] <= 8) == (waves == 1)
    cols = 64 if waves == 1 else 16
    assert k["launches"][1]["block"] == 64 * waves
    assert k["launches"][1]["grid"] >= -(-m // 4 + -cols + 1) // cols
