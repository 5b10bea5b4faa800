"""The additive predictor and the learned model's features describe the kernel that is
generated: a plan with nothing requested is priced in the environment that
kf_plan_kernel_params reports for it (all zero for row-stream kernels), in a table
without it as small workgroups, and its features hold its own geometry."""
import numpy as np
import pytest

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S

CG = kf.KF_COMPILE_CODEGEN_ONLY
KEYS = ("mat_k", "mat_waves", "mat_group", "mat_rows")


def entries(env, load):
    return [(1, env, 0, load), (1, env, 1, 1e-9), (1, env, 2, 1e-12), (1, env, 3, 1e-12), (1, env, 4, 1e-12), (1, env, 10, 0.0)]


def small_env(m, n):
    """Library defaults of a requested point: one float4 a lane, four waves, four rows a step."""
    r = -(-m // -(-2048 // -(-n // 256)))
    return (1, 4, 4, max(16, min(512, -(-r // 16) * 16)))


@pytest.mark.parametrize("seq,n", [("gemver", 16384), ("gemver", 3001), ("bicgk", 12001), ("bicgk", 2000), ("gesummv", 5003)])
def test_priced_in_its_own_environment(seq, n):
    q = S.by_name(seq, n, n, {"alpha": 1.5, "beta": 0.75})
    p = kf.kf_compile(q.script, mode="fused", flags=CG)
    par = kf.kf_plan_kernel_params(p, 0)
    own = tuple(par.get(k, 0) for k in KEYS)
    elsewhere = small_env(n, n)
    assert own != elsewhere
    extra = entries((0, 0, 0, 0), 3e-6) if own != (0, 0, 0, 0) else []     # a later row-stream kernel
    mine = kf.kf_predict_additive(p, kf.routine_table(entries(own, 3e-6) + entries(elsewhere, 1e-3) + extra))
    mats = 2 if seq == "gesummv" else 1
    passes = 2 if seq == "gemver" else 1
    assert mine == pytest.approx(mats * passes * n * n * 3e-6, rel=0.02)
    other = kf.kf_predict_additive(p, kf.routine_table(entries(elsewhere, 1e-3)))
    assert other == pytest.approx(mats * passes * n * n * 1e-3, rel=0.02)
    f = kf.kf_plan_features(p)[0]
    block = 2.0 ** f[24]
    assert f[17] * 64 == pytest.approx(block, rel=1e-3)                    # waves and workgroup agree
    if own != (0, 0, 0, 0):
        assert (f[16], f[17], 2.0 ** f[18], round(2.0 ** f[19])) == own
    kf.kf_plan_destroy(p)
