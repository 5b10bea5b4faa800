"""Kernels that store a matrix keep enough waves on the chip where it has few columns or
is quantised: rank-one updates alone take small workgroups below 1024 columns and for
BF16 and FP8 sources off 1 KiB boundaries, GEMVER's first kernel sixteen waves a CU
below 256 and for such sources."""
import json

import pytest

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S

CG = kf.KF_COMPILE_CODEGEN_ONLY


def kernels(mode, m, n):
    q = S.gemver(m, n, 1.5, 0.75)
    p = kf.kf_compile(q.script, mode=mode, flags=CG)
    d = json.loads(kf.kf_plan_describe(p))["kernels"]
    kf.kf_plan_destroy(p)
    return [k["params"] for k in d], [k["launches"][0] for k in d]


@pytest.mark.parametrize("n", [40, 100, 255, 300, 700, 1000])
def test_rank_one_updates_alone(n):
    prm, launch = kernels("unfused", 200000 if n < 256 else 60000, n)
    for k, l in list(zip(prm, launch))[:2]:
        assert (k["k"], k["waves"], k["group"]) == (1, 4, 4) and l["grid"] >= 1000, (k, l)


@pytest.mark.parametrize("n", [40, 100, 255])
def test_first_kernel_of_gemver(n):
    prm, launch = kernels("fused", 200000, n)
    assert prm[0]["k"] == 1 and launch[0]["grid"] * launch[0]["block"] >= 256 * 14 * 64, (prm[0], launch[0])


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("m,n", [(4001, 4000), (1058, 7500), (9001, 9000)])
def test_quantised_source_off_line_boundaries(dtype, m, n):
    q = S.gemver_q(m, n, 1.5, 0.75, dtype)
    p = kf.kf_compile(q.script, mode="fused", flags=CG)
    k = json.loads(kf.kf_plan_describe(p))["kernels"][0]
    kf.kf_plan_destroy(p)
    assert k["params"]["k"] == 1
    assert k["launches"][0]["grid"] * k["launches"][0]["block"] >= 256 * 14 * 64, k


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("m,n,small", [(4001, 4000, True), (2000, 8000, True), (9001, 9000, False), (4096, 4096, False)])
def test_quantised_rank_one_update_alone(dtype, m, n, small):
    q = S.gemver_q(m, n, 1.5, 0.75, dtype)
    p = kf.kf_compile(q.script, mode="unfused", flags=CG)
    k = json.loads(kf.kf_plan_describe(p))["kernels"][0]["params"]
    kf.kf_plan_destroy(p)
    assert (k["waves"] == 4) == small, k
