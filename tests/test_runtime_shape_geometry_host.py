"""A plan compiled for shapes up to a declared one takes small workgroups, whatever fills
the chip at the declared shape: a run at a smaller shape still has many row blocks."""
import pytest

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S


@pytest.mark.parametrize("seq", ["bicgk", "gemver", "sgemvt"])
@pytest.mark.parametrize("n", [500, 2048, 4096, 16384])
def test_small_workgroups(seq, n):
    q = S.by_name(seq, n, n, {"alpha": 1.5, "beta": 0.75})
    p = kf.kf_compile(q.script, mode="unfused", flags=kf.KF_COMPILE_CODEGEN_ONLY | kf.KF_COMPILE_RUNTIME_SHAPE)
    for k in range(kf.kf_plan_num_kernels(p)):
        par = kf.kf_plan_kernel_params(p, k)
        if par:                                        # row-stream kernels report nothing requested
            assert (par["mat_k"], par["mat_waves"], par["mat_group"]) == (1, 4, 4) and par["mat_rows"] <= 512, par
    kf.kf_plan_destroy(p)
