"""Requested strip points with several 16-byte units of BF16 or FP8 a step: the generated
kernel issues every load of a step before it waits for the first."""
import os
import re
import subprocess

import pytest

from paper_1305_1183_amd import build as B
from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S


@pytest.mark.parametrize("fmt,point", [("fp8", (2, 4, 2)), ("fp8", (1, 4, 4)), ("bf16", (2, 4, 4)), ("fp8", (2, 8, 2))])
def test_loads_before_the_first_wait(fmt, point, tmp_path):
    k, waves, group = point
    q = S.bicgk_q(16384, 16384, fmt)
    p = kf.kf_compile(q.script, mode="fused", flags=kf.KF_COMPILE_CODEGEN_ONLY, mat_k=k, mat_waves=waves, mat_group=group,
                      mat_rows=1024)
    src = "#include <hip/hip_runtime.h>\n" + open(os.path.join(B.CSRC, "device", "kf_blocks.h")).read() + kf.kf_plan_source(p, 0)
    kf.kf_plan_destroy(p)
    f = tmp_path / "k.hip"
    f.write_text(src)
    out = str(tmp_path / "k.s")
    subprocess.run([B.HIPCC, "-x", "hip"] + B.DEVICE + ["--cuda-device-only", "-O3", "-std=c++17", "-ffp-contract=off", "-S", str(f),
                    "-o", out], check=True, capture_output=True)
    body = open(out).read().split("_fin:")[0]
    most = 0
    for block in re.split(r"^\.LBB", body, flags=re.M):
        n = 0
        for line in block.splitlines():
            if re.search(r"global_load_dwordx4 .* nt", line):
                n += 1
            elif "s_waitcnt vmcnt" in line:
                n = 0
            most = max(most, n)
    assert most == k * group, (most, k * group)
