"""Where BF16 and FP8 kernels stream rows, and how many rows a wave shares."""
import json

import pytest

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S


def kernels(q, mode, **opts):
    p = kf.kf_compile(q.script, mode=mode, flags=kf.KF_COMPILE_CODEGEN_ONLY, **opts)
    d = json.loads(kf.kf_plan_describe(p))["kernels"]
    kf.kf_plan_destroy(p)
    return [k["params"] for k in d]


@pytest.mark.parametrize("fmt,m,n,stream,group", [
    ("fp8", 1500, 20000, False, 0), ("fp8", 1023, 20000, True, 1), ("fp8", 4096, 16384, True, 4), ("fp8", 4095, 16384, False, 0),
    ("fp8", 1500, 16383, True, 2), ("bf16", 1100, 30000, False, 0), ("bf16", 1500, 20000, True, 1), ("bf16", 2000, 8000, True, 1),
    ("bf16", 16384, 16384, True, 4)])
def test_gemv_alone(fmt, m, n, stream, group):
    p = kernels(S.bicgk_q(m, n, fmt), "unfused")[0]
    assert (p.get("schedule") == "row-stream") == stream, p
    if stream:
        assert p["group"] == group, p


@pytest.mark.parametrize("fmt,m,n,group", [("fp8", 16384, 16384, 2), ("bf16", 3000, 12000, 2), ("fp8", 2000, 8000, 1)])
def test_gemv_alone_in_units_of_four(fmt, m, n, group):
    p = kernels(S.bicgk_q(m, n, fmt), "unfused", mat_unit=4)[0]
    assert p["schedule"] == "row-stream" and p["group"] == group, p
