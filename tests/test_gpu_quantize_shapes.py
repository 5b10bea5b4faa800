"""The GPU row quantiser at the edges of its lane and register tiles, with rows
that start on any 4-byte boundary, wider padding, and rows that leave its fast
conversion (an infinity, NaN, a scale outside the fast range): every code and
scale equals the host quantiser's, which rounds the float64 quotient."""
import numpy as np
import pytest
import torch

from paper_1305_1183_amd import inputs as I
from paper_1305_1183_amd import kf
from paper_1305_1183_amd import quant as Q

pytestmark = pytest.mark.gpu

COLS = [1, 2, 3, 4, 5, 63, 255, 256, 257, 511, 512, 513, 1023, 1025, 2047, 2049, 4095, 4097, 8191, 8193, 16383, 16385,
        32767, 32769, 40000]


@pytest.mark.parametrize("fmt", ["bf16", "fp8"])
@pytest.mark.parametrize("cols", COLS)
def test_tile_edges(fmt, cols):
    rows, lda = 6, cols + cols % 3
    A = (I.normal(cols, 0, rows * cols).reshape(rows, cols)).astype(np.float32)
    A[1] *= np.float32(2.0 ** -110)                       # scale below the fast range
    A[2] *= np.float32(2.0 ** 110)                        # and above it
    A[3] = np.round(A[3] * 4)                             # exact ties and zeros
    A[3, 0] = 448.0
    A[4, cols // 2] = np.inf                              # scale 1, everything above 448 saturates
    A[5, cols - 1] = np.nan
    store = np.full((rows, lda), np.nan, np.float32)
    store[:, :cols] = A
    unit = 16 if fmt == "fp8" else 8
    ldq = (cols + unit - 1) // unit * unit + unit * (cols % 2)
    d = torch.from_numpy(store).cuda()
    codes = torch.full((rows, ldq), 0x5A, dtype=torch.uint8 if fmt == "fp8" else torch.int16, device="cuda")
    scales = torch.full((rows,), float("nan"), dtype=torch.float32, device="cuda")
    kf.kf_quantize_rows(d.data_ptr(), rows, cols, lda, kf.KF_FP8_E4M3 if fmt == "fp8" else kf.KF_BF16,
                        codes.data_ptr(), ldq, scales.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = codes.cpu().numpy().view(np.uint8 if fmt == "fp8" else np.uint16)
    amax = np.nanmax(np.where(np.isnan(A), 0, np.abs(A)), axis=1)
    want_s = np.ones(rows, np.float32)
    if fmt == "fp8":
        use = (amax > 0) & np.isfinite(amax)
        want_s[use] = amax[use] / np.float32(448.0)
    assert np.array_equal(scales.cpu().numpy().view(np.uint32), want_s.view(np.uint32))
    with np.errstate(invalid="ignore"):
        for r in range(rows):
            x = A[r].astype(np.float64)
            if fmt == "fp8":
                want = Q.to_e4m3_codes(np.clip(x / np.float64(want_s[r]), -1e30, 1e30))
            else:
                want = Q.to_bf16_codes(np.where(np.isnan(x), 0.0, x))
                want[np.isnan(x)] = got[r, :cols][np.isnan(x)]      # NaN payloads are checked on their own below
            assert np.array_equal(got[r, :cols], want), r
    if fmt == "bf16":
        assert got[5, cols - 1] & 0x7FFF > 0x7F80                   # still a NaN
    assert np.all(got[:, cols:] == 0)
