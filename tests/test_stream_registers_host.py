"""Row-stream kernels of several BF16 or FP8 matrices share x between as many rows as the
registers allow: none of them spills, and at least two waves a SIMD are left."""
import json
import os
import re
import subprocess

import pytest

from paper_1305_1183_amd import build as B
from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S


def products(m, n, fmts):
    """y = sum of A_i x, one kernel."""
    q = S._seq("products")
    x, one, y = S._vec(q, "x", n), S._const(q, "one", 1.0), None
    for i, f in enumerate(fmts):
        A = S._qmat(q, "A%d" % i, m, n, f)
        y = kf.kf_gemv(q.script, one, A, x, one, y) if y is not None else kf.kf_gemv(q.script, one, A, x)
    S._out(q, "y", y)
    return q


@pytest.mark.parametrize("fmts", [("fp8",) * 2 + ("f32",) * 3, ("fp8",) * 5, ("bf16",) * 5, ("fp8", "f32"), ("fp8", "bf16"),
                                  ("bf16",) * 2 + ("f32",) * 3, ("fp8", "f32", "f32")])
def test_no_spills(fmts, tmp_path):
    q = products(16384, 16384, fmts)
    p = kf.kf_compile(q.script, mode="fused", flags=kf.KF_COMPILE_CODEGEN_ONLY)
    kernels = json.loads(kf.kf_plan_describe(p))["kernels"]
    assert len(kernels) == 1 and kernels[0]["params"]["schedule"] == "row-stream"
    src = "#include <hip/hip_runtime.h>\n" + open(os.path.join(B.CSRC, "device", "kf_blocks.h")).read() + kf.kf_plan_source(p, 0)
    kf.kf_plan_destroy(p)
    f = tmp_path / "k.hip"
    f.write_text(src)
    r = subprocess.run([B.HIPCC, "-x", "hip"] + B.DEVICE + ["--cuda-device-only", "-O3", "-std=c++17", "-ffp-contract=off", "-c", str(f),
                        "-o", str(tmp_path / "k.o"), "-Rpass-analysis=kernel-resource-usage"], check=True, capture_output=True, text=True)
    assert re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr) == ["0"]
    assert int(re.findall(r"Occupancy \[waves/SIMD\]: (\d+)", r.stderr)[0]) >= 2, r.stderr
