"""Narrow row-resident kernels run in teams of one wave with 256 VGPRs a lane: the
register budget they are marked and ranked by is theirs, not that of 16 waves."""
import json

import pytest

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S

ENV = (0, 0, 0, 0)


@pytest.mark.parametrize("name,layout,widths", [("atax", kf.KF_ROW_MAJOR, (1000, 1281, 1500, 1800, 2047, 2048, 2049)),
                                                ("sgemvt", kf.KF_COL_MAJOR, (1500, 2048)),
                                                ("gemver", kf.KF_COL_MAJOR, (700, 768, 1000, 1200))])
def test_narrow_kernels_are_within_budget(name, layout, widths):
    T = kf.routine_table([(2, ENV, r, 1e-9, 0) for r in range(5)] + [(2, ENV, 10, 3.0, 0)])
    for w in widths:
        m, n = (30000, w) if layout == kf.KF_ROW_MAJOR else (w, 30000)
        q = S.by_name(name, m, n, {"alpha": 1.5, "beta": 0.75}, layout=layout)
        p = kf.kf_compile(q.script, mode="fused", flags=kf.KF_COMPILE_CODEGEN_ONLY)
        for k in json.loads(kf.kf_plan_describe(p))["kernels"]:
            assert k["params"]["teams"] == (8 if w <= 2048 else 1)
            assert not k["params"]["over_register_budget"], (name, w, k["params"])
        assert kf.kf_predict_additive(p, T) < 1e6, (name, w)
        kf.kf_plan_destroy(p)
