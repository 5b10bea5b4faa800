"""Column sums in the library's strip geometry: a wave's plain FP32 chain is no longer
than in the small workgroups (four waves, four rows a step, at most 512 rows) within 5%
of the error, the grid has no nearly empty second round, the workspace is no larger, and
a plan compiled again from the parameters it reports is the same kernel."""
import json

import pytest

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S

CG = kf.KF_COMPILE_CODEGEN_ONLY


def plan(seq, fmt, m, n, **kw):
    q = (S.by_name(seq, m, n, {"alpha": 1.5, "beta": 0.75}) if fmt == "f32" else
         S.bicgk_q(m, n, fmt) if seq == "bicgk" else S.gemver_q(m, n, 1.5, 0.75, fmt))
    p = kf.kf_compile(q.script, mode="fused", flags=CG, **kw)
    d = json.loads(kf.kf_plan_describe(p))["kernels"]
    par = [kf.kf_plan_kernel_params(p, k) for k in range(len(d))]
    ws = kf.kf_plan_workspace_bytes(p)
    kf.kf_plan_destroy(p)
    return d, par, ws


def small_workgroups(m, n, E):
    """Rows of the small workgroups' blocks."""
    strips = -(-n // (64 * E))
    r = -(-m // -(-2048 // strips))
    return max(16, min(512, -(-r // 16) * 16))


def chain_error(k, m):
    """Squared roundings per row (in units of one) of a wave's sum before pairs take over."""
    rows = -(-m // k["row_blocks"])
    G = k["group"]
    n = -(-rows // (k["waves"] * G)) * G
    if k["column_sums"] == "pairs":
        n = min(n, G)
    elif k["column_sums"] == "steps" and G > 1:
        return (G + 1) / 2 + n / (2 * G)
    return (n + 1) / 2


SHAPES = [(1024, 1024), (2448, 2448), (3000, 3000), (4096, 4096), (5003, 5003), (8192, 8192), (10007, 10007), (16384, 16384),
          (20000, 20000), (24000, 24000), (32768, 32768), (20000, 700), (300, 66000), (3000, 30000), (9000, 1500),
          (50000, 500), (100000, 90), (700, 16000), (9001, 9001), (3000, 20000), (40000, 4000)]


@pytest.mark.parametrize("fmt", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("seq", ["bicgk", "gemver"])
def test_chains_grid_and_workspace(seq, fmt):
    for m, n in SHAPES:
        d, par, ws = plan(seq, fmt, m, n)
        k = d[0]["params"]
        E = k["unit_elems"]
        few = small_workgroups(m, n, E)
        scaled = 1.0 if fmt != "f32" else 0.0            # the row scale is one more rounding
        assert chain_error(k, m) + scaled <= 1.11 * ((few / 4 + 1) / 2 + scaled), (seq, fmt, m, n, k)
        # one round of workgroups: 16 or 8 waves on a CU for FP32, up to 24 for the others
        grid = k["strips"] * -(-k["row_blocks"] // k["turns"])
        if m * n > 6e6:
            assert grid * k["waves"] <= 256 * (24 if E > 4 else 16) or k["strips"] > 256, (seq, fmt, m, n, k, grid)
            assert d[0]["launches"][0]["grid"] == grid
        base, _, base_ws = plan(seq, fmt, m, n, mat_k=1, mat_waves=4, mat_group=4, mat_rows=few)
        assert ws <= base_ws, (seq, fmt, m, n, ws, base_ws)


@pytest.mark.parametrize("fmt", ["f32", "fp8"])
@pytest.mark.parametrize("shape", [(24000, 24000), (20000, 700), (32768, 32768), (9000, 1500), (2448, 2448), (5003, 5003)], ids=str)
@pytest.mark.parametrize("seq", ["bicgk", "gemver"])
def test_reported_parameters_give_the_same_kernel(seq, shape, fmt):
    d, par, ws = plan(seq, fmt, *shape)
    again, _, ws2 = plan(seq, fmt, *shape, kernel_params=par)
    assert [k["launches"][0]["name"] for k in d] == [k["launches"][0]["name"] for k in again] and ws == ws2
