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


@pytest.mark.parametrize("fmt", ["bf16", "fp8"])
def test_units_of_a_stored_matrix_are_decoded_as_they_come(fmt):
    q = S.gemver_q(32768, 32768, 1.5, 0.75, fmt)
    p = kf.kf_compile(q.script, mode="fused", flags=kf.KF_COMPILE_CODEGEN_ONLY, mat_k=1, mat_waves=8, mat_group=4, mat_rows=256, mat_unit=16)
    src = kf.kf_plan_source(p, 0)
    kf.kf_plan_destroy(p)
    assert "sched_barrier" not in src and "kf_dec_%s(kf_ldu_nt(" % fmt in src
