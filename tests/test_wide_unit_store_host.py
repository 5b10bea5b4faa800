"""A matrix stored from FP8 in units of sixteen elements keeps the small workgroups where
larger blocks would need pairs."""
import json

import pytest

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S


def kernels(q, mode, **opts):
    p = kf.kf_compile(q.script, mode=mode, flags=kf.KF_COMPILE_CODEGEN_ONLY, **opts)
    d = json.loads(kf.kf_plan_describe(p))["kernels"]
    kf.kf_plan_destroy(p)
    return [k["params"] for k in d]


@pytest.mark.parametrize("fmt,n,small", [("fp8", 16384, True), ("fp8", 4096, True), ("bf16", 16384, False)])
def test_stored_matrix_in_wide_units(fmt, n, small):
    p = kernels(S.gemver_q(n, n, 1.5, 0.75, fmt), "fused", mat_unit=16)[0]
    assert (p["waves"] == 4) == small, p
