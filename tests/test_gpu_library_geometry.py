"""Kernels in the library's own geometry against the FP64 oracle (1e-5 log2 n): row
dots streamed by whole waves at the edges of strips, steps and shared rows, in every
storage format, with a fused rank-1 update and at run-time shapes; strip kernels on
both sides of the small-matrix line, with long row ranges; and the same bits fused and
unfused where both take the same geometry."""
import numpy as np
import pytest
import torch

import oracle
import seqcheck as SC
from oracle import quant as OQ
from paper_1305_1183_amd import inputs as I
from paper_1305_1183_amd import kf
from paper_1305_1183_amd import quant as Q
from paper_1305_1183_amd import sequences as S
from paper_1305_1183_amd import workloads as WL

pytestmark = pytest.mark.gpu

# (rows, cols): below, at and past one strip (256), steps of 8 strips, rows shared by two and
# four waves (fewer than 1024 rows; 8192 columns and more), four rows per wave
STREAM = [(1, 1), (5, 3), (3, 255), (9, 256), (9, 257), (2, 1030), (1025, 2047), (1100, 2049), (77, 4100), (1030, 8191),
          (1029, 8192), (1027, 10007), (40, 16385), (4099, 200), (5000, 256)]


@pytest.mark.parametrize("shape", STREAM, ids=str)
def test_streamed_row_dots(shape):
    m, n = shape
    for name in ("gesummv", "sgemvt"):
        arrays, scal = WL.make(name, m, n, seed=51)
        _, prog, host = SC.run_gpu(name, m, n, arrays, scal)
        SC.check_against_oracle(name, m, n, host, SC.oracle_outputs(name, arrays, scal, n))
        assert prog.describe()["kernels"][-1]["params"]["schedule"] == "row-stream"


@pytest.mark.parametrize("fmt", ["bf16", "fp8"])
@pytest.mark.parametrize("shape", [(3, 17), (70, 511), (70, 1025), (1030, 2060), (1100, 9001), (1026, 16400)], ids=str)
def test_streamed_quantised_row_dots(shape, fmt):
    """gemv of a quantised matrix beside the same matrix in FP32 (one kernel each and both in one)."""
    m, n = shape
    st, sc = Q.quantize_rows(I.normal(52, 0, m * n).reshape(m, n), fmt)
    A32 = I.matrix(52, 1, m, n, ld=I.padded_ld(n))
    x = I.vector(52, 2, n)
    deq = OQ.decode_bf16(st) if fmt == "bf16" else OQ.decode_e4m3(st)
    deq = deq[:, :n] * sc.astype(np.float64)[:, None]
    ref = deq @ x + 0.5 * (A32[:, :n].astype(np.float64) @ x)
    q = S._seq("mixed")
    A = S._qmat(q, "A", m, n, fmt)
    B = S._mat(q, "B", m, n)
    xv = S._vec(q, "x", n)
    one, half = S._const(q, "one", 1.0), S._const(q, "half", 0.5)
    t = kf.kf_gemv(q.script, one, A, xv)
    S._out(q, "y", kf.kf_gemv(q.script, half, B, xv, one, t))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a.view(np.int16) if a.dtype == np.uint16 else a)).cuda()
    for mode in ("fused", "unfused"):
        out = q.compile(mode).bind(A=dev(st), A_scale=dev(sc), B=dev(A32), x=dev(x)).run()
        assert WL.rel_l2(out["y"].cpu().numpy(), ref) <= WL.tolerance("gesummv", m, n), mode


@pytest.mark.parametrize("keep", [False, True], ids=["dropped", "stored"])
@pytest.mark.parametrize("shape", [(6, 250), (300, 1030), (1025, 8200)], ids=str)
def test_streamed_rank_one_update(shape, keep):
    """y = (A + u v^T) x in one kernel, with the updated matrix kept on chip or stored."""
    m, n = shape
    q = S._seq("ger_gemv")
    A, u, v, x = S._mat(q, "A", m, n), S._vec(q, "u", m), S._vec(q, "v", n), S._vec(q, "x", n)
    one = S._const(q, "one", 1.0)
    B = kf.kf_ger(q.script, one, A, u, v)
    if keep:
        S._out(q, "B", B)
    S._out(q, "y", kf.kf_gemv(q.script, one, B, x))
    a = {"A": I.matrix(53, 0, m, n, ld=I.padded_ld(n)), "u": I.vector(53, 1, m), "v": I.vector(53, 2, n), "x": I.vector(53, 3, n)}
    prog = q.compile("fused").bind(**{k: torch.from_numpy(t).cuda() for k, t in a.items()})
    assert prog.num_kernels == 1
    out = {k: t.cpu().numpy() for k, t in prog.run().items()}
    Bref = a["A"][:, :n].astype(np.float64) + np.outer(a["u"].astype(np.float64), a["v"])
    assert WL.rel_l2(out["y"], Bref @ a["x"]) <= WL.tolerance("gesummv", m, n)
    if keep:
        assert WL.rel_l2(out["B"][:, :n], Bref) <= 1e-6


@pytest.mark.parametrize("shape", [(130, 70), (511, 512), (1, 3), (512, 512)], ids=str)
def test_streamed_run_time_shape(shape):
    m, n = shape
    q = S.sgemvt(512, 512, 1.5, 0.5) if m == n else S.sgemvt(512, 513, 1.5, 0.5)
    plan = kf.kf_compile(q.script, mode="fused", flags=kf.KF_COMPILE_RUNTIME_SHAPE)
    kf.kf_plan_set_shape(plan, m, n)
    ld = I.padded_ld(n) + 4
    a = {"A": I.matrix(54, 0, m, n, ld=ld), "y": I.vector(54, 1, m), "z": I.vector(54, 2, n)}
    dev = {k: torch.from_numpy(t).cuda() for k, t in a.items()}
    kf.kf_bind_matrix(plan, q.values["A"], dev["A"].data_ptr(), ld)
    x, w = torch.empty(n, device="cuda"), torch.empty(m, device="cuda")
    for name, t in (("y", dev["y"]), ("z", dev["z"]), ("x", x), ("w", w)):
        kf.kf_bind(plan, q.values[name], t.data_ptr())
    need = kf.kf_plan_workspace_bytes(plan)
    ws = torch.empty(need // 4 + 64, device="cuda")
    kf.kf_bind_workspace(plan, (ws.data_ptr() + 255) // 256 * 256, need)
    kf.kf_run(plan, torch.cuda.current_stream().cuda_stream)
    rx, rw = oracle.sgemvt(1.5, 0.5, a["A"], a["y"], a["z"], cols=n)
    assert WL.rel_l2(x.cpu().numpy(), rx) <= WL.tolerance("sgemvt", m, n)
    assert WL.rel_l2(w.cpu().numpy(), rw) <= WL.tolerance("sgemvt", m, n)
    kf.kf_plan_destroy(plan)


# both sides of six million elements, aligned and ragged columns, few rows and few columns
STRIP = [(2448, 2450), (2451, 2450), (2500, 2560), (20000, 301), (9000, 700), (300, 20003), (17000, 513)]


@pytest.mark.parametrize("shape", STRIP, ids=str)
def test_strip_geometry(shape):
    m, n = shape
    for name in ("bicgk", "gemver"):
        arrays, scal = WL.make(name, m, n, seed=55)
        _, _, host = SC.run_gpu(name, m, n, arrays, scal)
        SC.check_against_oracle(name, m, n, host, SC.oracle_outputs(name, arrays, scal, n))


@pytest.mark.parametrize("rows", [128, 129, 130, 400])
def test_long_row_ranges(rows):
    """One wave per block of `rows` rows: its column sums are carried in pairs past 128 rows."""
    m, n = 777, 300
    arrays, scal = WL.make("gemver", m, n, seed=56)
    _, _, host = SC.run_gpu("gemver", m, n, arrays, scal, mat_k=1, mat_waves=1, mat_group=1, mat_rows=rows)
    SC.check_against_oracle("gemver", m, n, host, SC.oracle_outputs("gemver", arrays, scal, n))


@pytest.mark.parametrize("shape", [(1030, 5003), (3000, 2500), (700, 9000)], ids=str)
def test_fused_and_unfused_give_the_same_bits(shape):
    m, n = shape
    for name in ("bicgk", "gesummv"):
        arrays, scal = WL.make(name, m, n, seed=57)
        _, _, hf = SC.run_gpu(name, m, n, arrays, scal, mode="fused")
        _, _, hu = SC.run_gpu(name, m, n, arrays, scal, mode="unfused")
        for k in hf:
            assert np.array_equal(hf[k], hu[k]), (name, k)


def test_kernels_of_many_operands_still_compile():
    """Five column and five row reductions of two matrices and a rank-1 update in one kernel: the
    library's geometry gives way to small workgroups instead of outgrowing registers or LDS."""
    m, n = 3000, 2600
    q = S._seq("many")
    A, B = S._mat(q, "A", m, n), S._mat(q, "B", m, n)
    one = S._const(q, "one", 1.0)
    rng = {}
    for i in range(5):
        rng["x%d" % i], rng["r%d" % i] = I.vector(58, i, n), I.vector(58, 10 + i, m)
        xv, rv = S._vec(q, "x%d" % i, n), S._vec(q, "r%d" % i, m)
        S._out(q, "q%d" % i, kf.kf_gemv(q.script, one, A if i % 2 else B, xv))
        S._out(q, "s%d" % i, kf.kf_gemtv(q.script, one, B if i % 2 else A, rv))
    a = dict(rng, A=I.matrix(58, 20, m, n), B=I.matrix(58, 21, m, n))
    prog = q.compile("fused").bind(**{k: torch.from_numpy(t).cuda() for k, t in a.items()})
    out = {k: t.cpu().numpy() for k, t in prog.run().items()}
    mats = {k: a[k].astype(np.float64) for k in "AB"}
    for i in range(5):
        assert WL.rel_l2(out["q%d" % i], mats["A" if i % 2 else "B"] @ rng["x%d" % i]) <= 1.2e-4
        assert WL.rel_l2(out["s%d" % i], mats["B" if i % 2 else "A"].T @ rng["r%d" % i]) <= 1.2e-4
