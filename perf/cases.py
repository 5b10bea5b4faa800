"""Performance cases: the work that users of the library have it do, through its
public entry points, with an independent 64-bit reference of every result.

``listed()`` names one case per path and size class; ``draw(rng)`` gives one more
case of the same ranges. ``prepare(case, seed)`` holds what a program has before
the call (device inputs, the compiled plan and its buffers, the batch, the
network's parameters), ``run(state)`` is one pass, ``work(case)`` the bytes and
operations the pass cannot do without, and ``exact(case, seed)`` the results of
the same inputs in float64, from plain torch.

Plans are compiled as a program without a tuning step does: the fewest-kernel
partition with the library's own geometry for the shape.
"""
from __future__ import annotations

import math

import torch

from paper_1305_1183_amd import kf
from paper_1305_1183_amd import sequences as S
from paper_1305_1183_amd.batched import BICGK, INPUTS, OUTPUTS, Batch, make_instances

DEV = "cuda"

# operands by sequence: (matrices, row-indexed vectors, column-indexed vectors)
OPERANDS = {
    "bicgk": (["A"], ["r"], ["p"]),
    "atax": (["A"], [], ["x"]),
    "gesummv": (["A", "B"], [], ["x"]),
    "gemver": (["A"], ["u1", "u2", "y"], ["v1", "v2", "z"]),
    "sgemvt": (["A"], ["y"], ["z"]),
}
VECTORS = {"axpydot": ["w", "v", "u"], "waxpby": ["x", "y"], "vadd": ["w", "y", "z"]}
# element bytes and row granularity (elements per 16 bytes) of matrix storage
STORAGE = {"f32": (4, 4), "bf16": (2, 8), "fp8": (1, 16)}


def listed():
    return [
        # a small solver's BiCG step: the parity problem, a few microseconds of work
        {"name": "bicgk-1024", "kind": "seq", "seq": "bicgk", "m": 1024, "n": 1024, "layout": "row", "fmt": "f32"},
        # a vector update of an iterative method on an odd-sized grid
        {"name": "waxpby-1000003", "kind": "vec", "seq": "waxpby", "n": 1000003},
        # the benchmark's vector length: update and dot product in one pass
        {"name": "axpydot-2^26", "kind": "vec", "seq": "axpydot", "n": 1 << 26},
        # the benchmark's matrix size: one read of A for A p and A^T r
        {"name": "bicgk-16384", "kind": "seq", "seq": "bicgk", "m": 16384, "n": 16384, "layout": "row", "fmt": "f32"},
        # the normal-equations product of a tall least-squares matrix
        {"name": "atax-30011x1021", "kind": "seq", "seq": "atax", "m": 30011, "n": 1021, "layout": "row", "fmt": "f32"},
        # two dense operators of an ordinary, odd size applied to one vector
        {"name": "gesummv-5003", "kind": "seq", "seq": "gesummv", "m": 5003, "n": 5003, "layout": "row", "fmt": "f32"},
        # the benchmark's largest sequence: a rank-2 update that is stored and used twice
        {"name": "gemver-16384", "kind": "seq", "seq": "gemver", "m": 16384, "n": 16384, "layout": "row", "fmt": "f32"},
        # the same sequence on the column-major matrix of a Fortran or BLAS program
        {"name": "gemver-col-8192", "kind": "seq", "seq": "gemver", "m": 8192, "n": 8192, "layout": "col", "fmt": "f32"},
        # reduced-precision storage of a matrix that is applied many times
        {"name": "bicgk-fp8-16384", "kind": "seq", "seq": "bicgk", "m": 16384, "n": 16384, "layout": "row", "fmt": "fp8"},
        # producing that storage from the FP32 matrix
        {"name": "quantize-fp8-8192", "kind": "quantize", "m": 8192, "n": 8192, "fmt": "fp8"},
        # many small independent problems of mixed sizes in one launch
        {"name": "batch-512+512", "kind": "batch", "bicgk": 512, "gemver": 512, "lo": 32, "hi": 2048, "sizes": 1},
        # one optimiser step of the plan-ranking network at its training batch
        {"name": "mlp-step-256", "kind": "mlp", "d": 32, "h": 128, "layers": 3, "n": 256},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    """One more case: a path by its share of use, sizes spread over the logarithm."""
    path = rng.choices(["vec", "seq", "col", "prec", "quantize", "batch", "mlp"], [3, 6, 2, 2, 2, 2, 1])[0]
    if path == "vec":
        return {"kind": "vec", "seq": rng.choice(sorted(VECTORS)), "n": _log(rng, 1 << 10, 1 << 26)}
    if path == "batch":
        total = _log(rng, 8, 1024)
        b = rng.randint(0, total)
        lo = _log(rng, 1, 256)
        return {"kind": "batch", "bicgk": b, "gemver": total - b, "lo": lo, "hi": rng.randint(lo, 2048),
                "sizes": rng.randint(1, 1 << 20)}
    if path == "mlp":
        return {"kind": "mlp", "d": 32, "h": rng.choice([32, 64, 128, 200]), "layers": rng.randint(1, 4),
                "n": _log(rng, 16, 4096)}
    m = _log(rng, 64, 32768)
    n = m if m <= 16384 and rng.random() < 0.5 else _log(rng, 64, min(16384, (1 << 28) // m))
    if path == "quantize":
        # the largest listed case of this path moves 0.3 GB
        return {"kind": "quantize", "m": m, "n": max(64, min(n, (1 << 26) // m)), "fmt": rng.choice(["bf16", "fp8"])}
    if path == "prec":
        return {"kind": "seq", "seq": rng.choice(["bicgk", "gemver"]), "m": m, "n": n, "layout": "row",
                "fmt": rng.choice(["bf16", "fp8"])}
    if path == "col":
        return {"kind": "seq", "seq": rng.choice(["bicgk", "atax", "sgemvt", "gemver"]), "m": m, "n": n,
                "layout": "col", "fmt": "f32"}
    return {"kind": "seq", "seq": rng.choice(sorted(OPERANDS)), "m": m, "n": n, "layout": "row", "fmt": "f32"}


# ---- inputs --------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _uniform(g, *shape):
    return torch.empty(*shape, dtype=torch.float32, device=DEV).uniform_(-1.0, 1.0, generator=g)


def _scalars(seed):
    """alpha and beta, uniform on [0.5, 2)."""
    g = torch.Generator().manual_seed(int(seed))
    a, b = (0.5 + 1.5 * torch.rand(2, generator=g, dtype=torch.float32)).tolist()
    return {"alpha": a, "beta": b}


def _ld(cols, fmt):
    unit = STORAGE[fmt][1]
    return (cols + unit - 1) // unit * unit


def _store(g, rows, cols, fmt):
    """N(0, 1) rows stored as `fmt` with one scale per row: (codes, scales)."""
    codes = torch.zeros(rows, _ld(cols, fmt), dtype=torch.int16 if fmt == "bf16" else torch.uint8, device=DEV)
    scales = torch.ones(rows, dtype=torch.float32, device=DEV)
    for r in range(0, rows, 2048):
        x = torch.empty(min(2048, rows - r), cols, dtype=torch.float32, device=DEV).normal_(generator=g)
        if fmt == "bf16":
            codes[r:r + 2048, :cols] = x.to(torch.bfloat16).view(torch.int16)
        else:
            s = x.abs().amax(1) / 448.0
            codes[r:r + 2048, :cols] = (x / s[:, None]).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
            scales[r:r + 2048] = s
    return codes, scales


def _seq_inputs(case, seed):
    """Device operands by name; a column-major matrix is its cols x ld storage."""
    g = _gen(seed)
    m, n = case["m"], case["n"]
    mats, rowv, colv = OPERANDS[case["seq"]]
    t = {}
    for name in mats:
        if case["fmt"] != "f32":
            t[name], scale = _store(g, m, n, case["fmt"])
            t[name + "_scale"] = scale
        elif case["layout"] == "col":
            t[name] = _uniform(g, n, _ld(m, "f32"))
        else:
            t[name] = _uniform(g, m, _ld(n, "f32"))
    for name in rowv:
        t[name] = _uniform(g, m)
    for name in colv:
        t[name] = _uniform(g, n)
    return t


def _build(case, sc):
    if case["kind"] == "vec":
        return S.by_name(case["seq"], case["n"], case["n"], sc)
    if case["fmt"] != "f32":
        if case["seq"] == "bicgk":
            return S.bicgk_q(case["m"], case["n"], case["fmt"])
        return S.gemver_q(case["m"], case["n"], sc["alpha"], sc["beta"], case["fmt"])
    layout = kf.KF_COL_MAJOR if case["layout"] == "col" else kf.KF_ROW_MAJOR
    return S.by_name(case["seq"], case["m"], case["n"], sc, layout=layout)


def _mlp_inputs(case, seed):
    g = _gen(seed)
    d, h, L, n = case["d"], case["h"], case["layers"], case["n"]
    net = kf.kf_mlp_create(d, h, L)
    count = kf.kf_mlp_param_count(net)
    lay = [kf.kf_mlp_layout(net, l) for l in range(L + 1)]
    params = torch.from_numpy(kf.kf_mlp_init_params(net, int(seed))).to(DEV)
    X = torch.empty(n, d, device=DEV).normal_(generator=g)
    y = torch.empty(n, device=DEV).normal_(generator=g)
    # moments of a network in training
    m1 = 1e-3 * torch.empty(count, device=DEV).normal_(generator=g)
    m2 = 1e-6 * (0.5 + torch.empty(count, device=DEV).uniform_(0.0, 1.0, generator=g))
    return net, lay, params, X, y, m1, m2


# ---- one pass --------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind in ("vec", "seq"):
        if kind == "vec":
            g = _gen(seed)
            t = {name: _uniform(g, case["n"]) for name in VECTORS[case["seq"]]}
        else:
            t = _seq_inputs(case, seed)
        q = _build(case, _scalars(seed))
        # outputs with padded rows start defined, as the padding is never written
        outs = {name: torch.zeros(q.shapes[name], dtype=torch.float32, device=DEV) for name in q.outputs}
        return q.compile("fused").bind(**t, **outs).run
    if kind == "quantize":
        m, n = case["m"], case["n"]
        A = torch.empty(m, n, dtype=torch.float32, device=DEV).normal_(generator=_gen(seed))
        dtype, ldq = (kf.KF_BF16, kf.KF_FP8_E4M3)[case["fmt"] == "fp8"], _ld(n, case["fmt"])
        codes = torch.zeros(m, ldq, dtype=torch.int16 if case["fmt"] == "bf16" else torch.uint8, device=DEV)
        scales = torch.zeros(m, dtype=torch.float32, device=DEV)

        def quantize():
            kf.kf_quantize_rows(A.data_ptr(), m, n, n, dtype, codes.data_ptr(), ldq, scales.data_ptr(),
                                torch.cuda.current_stream().cuda_stream)
            return {"codes": codes, "scales": scales}
        return quantize
    if kind == "batch":
        b = Batch(*_instances(case))
        b.arena = _arena(b, seed)
        b.ws = torch.empty(max(256, b.ws_bytes), dtype=torch.uint8, device=DEV)
        kf.kf_batch_bind(b.h, b.arena.data_ptr(), b.ws.data_ptr(), b.stream())
        # the whole arena, and the vectors of instances spread over the batch by name
        out = {"arena": b.arena, **_spread(b, b.arena)}

        def batch():
            b.run()
            return out
        return batch
    net, lay, params, X, y, m1, m2 = _mlp_inputs(case, seed)
    grads, loss = torch.zeros_like(params), torch.zeros(1, device=DEV)
    nb = kf.kf_mlp_workspace_bytes(net, case["n"])
    ws = torch.empty(nb // 4 + 64, dtype=torch.float32, device=DEV)

    def step():
        st = torch.cuda.current_stream().cuda_stream
        kf.kf_mlp_loss_grad(net, params.data_ptr(), X.data_ptr(), y.data_ptr(), case["n"], grads.data_ptr(),
                            loss.data_ptr(), ws.data_ptr(), nb, st)
        kf.kf_mlp_adam(net, params.data_ptr(), grads.data_ptr(), m1.data_ptr(), m2.data_ptr(), 100, 1e-3, stream=st)
        return {"loss": loss, "grads": grads, "params": params, "m1": m1, "m2": m2}
    return step


def run(state):
    return state()


# ---- the batch -------------------------------------------------------------------
def _instances(case):
    return make_instances(case["bicgk"], case["gemver"], case["sizes"], case["lo"], case["hi"])


def _arena(b, seed):
    """Every operand uniform on [-1, 1); what is an output is overwritten."""
    return _uniform(_gen(seed), max(1, b.elems))


def _spread(b, arena):
    out = {}
    count = len(b.kinds)
    for i in sorted({j * (count - 1) // 23 for j in range(24)}):
        for name in OUTPUTS[int(b.kinds[i])]:
            off, _ = b.offset(i, name)
            out["%s%d" % (name, i)] = arena[off:off + int(b.ns[i])]
    return out


# ---- what a pass cannot do without --------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "vec":
        n = case["n"]
        vectors, flops = {"axpydot": (4, 4), "waxpby": (3, 3), "vadd": (4, 2)}[case["seq"]]
        return {"bytes": 4 * vectors * n, "flops": flops * n}
    if kind == "seq":
        m, n, seq = case["m"], case["n"], case["seq"]
        mats, rowv, colv = OPERANDS[seq]
        outm, outr, outc = {"bicgk": (0, 1, 1), "atax": (0, 0, 1), "gesummv": (0, 1, 0), "gemver": (1, 1, 1),
                            "sgemvt": (0, 1, 1)}[seq]
        es = STORAGE[case["fmt"]][0]
        byt = len(mats) * m * n * es + outm * m * n * 4 + 4 * ((len(rowv) + outr) * m + (len(colv) + outc) * n)
        return {"bytes": byt + (4 * m if es < 4 else 0), "flops": (8 if seq == "gemver" else 4) * m * n}
    if kind == "quantize":
        m, n = case["m"], case["n"]
        return {"bytes": m * n * (4 + STORAGE[case["fmt"]][0]) + 4 * m, "flops": 3 * m * n}
    if kind == "batch":
        kinds, ns, _, _ = _instances(case)
        byt = flops = 0
        for k, n in zip(kinds.tolist(), ns.tolist()):
            byt += 4 * (n * n + 4 * n) if k == BICGK else 4 * (2 * n * n + 8 * n)
            flops += (4 if k == BICGK else 8) * n * n
        return {"bytes": byt, "flops": flops}
    d, h, L, n = case["d"], case["h"], case["layers"], case["n"]
    weights = d * h + (L - 1) * h * h + h
    return {"bytes": 4 * (n * (d + 1) + 7 * (weights + L * h + 1)), "flops": 6 * weights * n}


# ---- 64-bit reference -----------------------------------------------------------------
def _bicgk(A, p, r):
    return A @ p, A.t() @ r


def _gemver(A, u1, v1, u2, v2, y, z, alpha, beta):
    B = A + torch.outer(u1, v1) + torch.outer(u2, v2)
    x = beta * (B.t() @ y) + z
    return B, x, alpha * (B @ x)


def exact(case, seed):
    kind = case["kind"]
    sc = _scalars(seed)
    a, b = sc["alpha"], sc["beta"]
    if kind == "vec":
        g = _gen(seed)
        t = {name: _uniform(g, case["n"]).double() for name in VECTORS[case["seq"]]}
        if case["seq"] == "axpydot":
            z = t["w"] - a * t["v"]
            return {"z": z, "r": (z * t["u"]).sum().reshape(1)}
        if case["seq"] == "waxpby":
            return {"w": a * t["x"] + b * t["y"]}
        return {"x": t["w"] + t["y"] + t["z"]}
    if kind == "seq":
        m, n, seq = case["m"], case["n"], case["seq"]
        raw = _seq_inputs(case, seed)
        t = {k: v.double() for k, v in raw.items() if v.dim() == 1}
        for k, v in raw.items():
            if v.dim() == 1:
                continue
            if case["fmt"] != "f32":
                code = v[:, :n].contiguous().view(torch.bfloat16 if case["fmt"] == "bf16" else torch.float8_e4m3fn)
                t[k] = code.float().double() * t[k + "_scale"][:, None]
            else:
                t[k] = v[:, :m].t().double() if case["layout"] == "col" else v[:, :n].double()
        A = t["A"]
        if seq == "bicgk":
            q, s = _bicgk(A, t["p"], t["r"])
            return {"q": q, "s": s}
        if seq == "atax":
            return {"y": A.t() @ (A @ t["x"])}
        if seq == "gesummv":
            return {"y": a * (A @ t["x"]) + b * (t["B"] @ t["x"])}
        if seq == "sgemvt":
            x = b * (A.t() @ t["y"]) + t["z"]
            return {"x": x, "w": a * (A @ x)}
        B, x, w = _gemver(A, *(t[k] for k in ("u1", "v1", "u2", "v2", "y", "z")), a, b)
        if case["layout"] == "col":
            B = B.t()
        padded = torch.zeros(B.shape[0], _ld(B.shape[1], "f32"), dtype=torch.float64, device=DEV)
        padded[:, :B.shape[1]] = B
        return {"B": padded, "x": x, "w": w}
    if kind == "quantize":
        A = torch.empty(case["m"], case["n"], dtype=torch.float32, device=DEV).normal_(generator=_gen(seed))
        s = A.abs().amax(1).double() / 448.0 if case["fmt"] == "fp8" else torch.ones(case["m"], dtype=torch.float64)
        return {"codes": None, "scales": s}
    if kind == "batch":
        kinds, ns, alpha, beta = _instances(case)
        b = Batch(kinds, ns, alpha, beta)     # only for the places of the operands in the arena
        arena = _arena(b, seed).double()

        def at(i, name):
            off, ld = b.offset(i, name)
            n = int(ns[i])
            return arena[off:off + n * ld].view(n, ld)[:, :n] if name in ("A", "B") else arena[off:off + n]
        for i, k in enumerate(kinds.tolist()):
            t = [at(i, "A")] + [at(i, name) for name in INPUTS[k]]
            if k == BICGK:
                res = dict(zip(("q", "s"), _bicgk(*t)))
            else:
                res = dict(zip(("B", "x", "w"), _gemver(*t, float(alpha[i]), float(beta[i]))))
            for name, v in res.items():
                at(i, name).copy_(v)
        return {"arena": arena, **_spread(b, arena)}
    net, lay, params, X, y, m1, m2 = _mlp_inputs(case, seed)
    kf.kf_mlp_destroy(net)
    p = params.double().requires_grad_(True)
    v = X.double()
    for l, (w, bias, rows, cols) in enumerate(lay):
        v = v @ p[w:w + rows * cols].view(rows, cols) + p[bias:bias + cols]
        v = v.relu() if l < len(lay) - 1 else v
    loss = (v[:, 0] - y.double()).square().mean()
    loss.backward()
    g = p.grad
    m1, m2 = 0.9 * m1.double() + 0.1 * g, 0.999 * m2.double() + 0.001 * g * g
    q = p.detach() - 1e-3 * (m1 / (1 - 0.9 ** 100)) / ((m2 / (1 - 0.999 ** 100)).sqrt() + 1e-8)
    return {"loss": loss.detach().reshape(1), "grads": g, "params": q, "m1": m1, "m2": m2}
