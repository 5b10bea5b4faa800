"""A matrix whose rows take 1024 lanes each and more than 2^32 threads together goes to
the GPU in several launches: the rows on both sides of the seam and the last ones get
the codes and scales that a launch of their own gives them."""
import pytest
import torch

from paper_1305_1183_amd import kf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["fp8", "bf16"])
def test_more_threads_than_a_launch_takes(fmt):
    rows, cols = 4194303 + 3, 8193
    unit, es = (16, 1) if fmt == "fp8" else (8, 2)
    ldq = (cols + unit - 1) // unit * unit
    need = rows * (cols * 4 + ldq * es + 4) + (4 << 30)
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip("needs %d GB of free device memory" % (need >> 30))
    print("case quantize limit", fmt, rows, cols, flush=True)
    dt, code = (kf.KF_FP8_E4M3, torch.uint8) if fmt == "fp8" else (kf.KF_BF16, torch.int16)
    A = torch.empty(rows, cols, device="cuda")
    codes = torch.empty(rows, ldq, dtype=code, device="cuda")
    scales = torch.empty(rows, device="cuda")
    seam = list(range(4194300, rows))
    g = torch.Generator(device="cuda").manual_seed(9)
    pick = [0, 1, 2] + seam
    for i in pick:
        A[i].normal_(generator=g)
        scales[i], codes[i] = -1.0, 5
    st = torch.cuda.current_stream().cuda_stream
    kf.kf_quantize_rows(A.data_ptr(), rows, cols, cols, dt, codes.data_ptr(), ldq, scales.data_ptr(), st)
    own = torch.zeros(len(pick), ldq, dtype=code, device="cuda")
    osc = torch.zeros(len(pick), device="cuda")
    part = A[pick].contiguous()
    kf.kf_quantize_rows(part.data_ptr(), len(pick), cols, cols, dt, own.data_ptr(), ldq, osc.data_ptr(), st)
    torch.cuda.synchronize()
    assert torch.equal(codes[pick], own) and torch.equal(scales[pick], osc)
    del A, codes, scales
    torch.cuda.empty_cache()
