"""Workloads of the checksum-protected products, one pass each through the
public entry points, for timing two versions of the library against each other.

A pass is what a program that relies on the protection does: encode the
operands (quantizing them first for bfloat16 and FP8), multiply, verify, and
act on the report -- so most passes end with the host reading the report, as
abft.Protected.verify does.  Inputs are the random dense matrices of this
repository's benchmark (uniform on [-1, 1)).

  listed()              the named cases
  draw(rng)             another case of the same ranges
  prepare(case, seed)   inputs, buffers and plans, on the GPU
  run(state)            one pass; returns everything it wrote
  exact(case, seed)     the same outputs in binary64 by plain torch
  work(case)            bytes and flops one pass cannot do without

The max |residual| / threshold ratios of the reports are left out of the
outputs: they are the rounding noise of the product itself.
"""
import numpy as np
import torch

from paper_0806_3121_amd import abft

DTYPES = {"f64": abft.ABFT_F64, "f32": abft.ABFT_F32, "bf16": abft.ABFT_BF16, "fp8": abft.ABFT_FP8_E4M3}
SIZE = {"f64": 8, "f32": 4, "bf16": 2, "fp8": 1}
REPORT_WORDS = 6        # n_flag_c, n_flag_r, n_excl_c, n_excl_r, n_nonfinite, status


def _step(name, dtype, m, n, k, br, bc, fused=False, rebuild=False, correct=False):
    c = {"kind": "step", "dtype": dtype, "m": m, "n": n, "k": k, "br": br, "bc": bc, "fused": fused,
         "rebuild": rebuild, "correct": correct}
    return dict(c, name=name) if name else c


def _panels(name, m, n, k, b, panels):
    c = {"kind": "panels", "m": m, "n": n, "k": k, "b": b, "panels": panels}
    return dict(c, name=name) if name else c


def _weighted(name, dtype, m, n, k, b, f):
    c = {"kind": "weighted", "dtype": dtype, "m": m, "n": n, "k": k, "b": b, "f": f}
    return dict(c, name=name) if name else c


def _batch(name, count, hi, br, shapes_seed):
    c = {"kind": "batch", "count": count, "lo": 64, "hi": hi, "step": 32, "br": br, "shapes_seed": shapes_seed}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest protected product anyone calls: launches and latency
        _step("f64_256_b1", "f64", 256, 256, 256, 1, 1),
        # the same with block checksums, one lost block rebuilt
        _step("f64_256_b64_rebuild", "f64", 256, 256, 256, 64, 64, rebuild=True),
        # sizes that fit no tile and an inner size that fits no slab, one located element corrected
        _step("f64_ragged_b1_correct", "f64", 2001, 1503, 1234, 1, 1, correct=True),
        # the default benchmark: an 8 x 8 grid of blocks, one of them lost and rebuilt
        _step("f64_8192_b1024_rebuild", "f64", 8192, 8192, 8192, 1024, 1024, rebuild=True),
        # binary32 with the statistical thresholds, long inner dimension
        _step("f32_8192x4096x16384_b1", "f32", 8192, 4096, 16384, 1, 1),
        # the large bfloat16 product, from binary32 operands
        _step("bf16_16384_b1", "bf16", 16384, 16384, 16384, 1, 1),
        # a ragged bfloat16 layer-sized product, verified from the product's own partial sums
        _step("bf16_ragged_b1_fused", "bf16", 3000, 5003, 2056, 1, 1, fused=True),
        # a large FP8 product, from binary32 operands
        _step("fp8_8192_b1", "fp8", 8192, 8192, 8192, 1, 1),
        # outer-product form: rank-256 updates, a block lost and rebuilt half-way
        _panels("f64_panels_2048_b256", 2048, 2048, 2048, 256, 8),
        # two weighted checksums, two blocks of one block column lost at once
        _weighted("f64_weighted_4096_b512_f2", "f64", 4096, 4096, 4096, 512, 2),
        # protected matrix-vector product: the weighted problem with one column
        {"kind": "matvec", "m": 16384, "k": 16384, "b": 512, "f": 2, "name": "f64_matvec_16384_f2"},
        # many independent uneven bfloat16 products in one pass (batch benchmark shapes)
        _batch("bf16_batch_512", 512, 2048, 32, 20080523),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _draw_step(rng):
    dtype = rng.choice(["f64", "f64", "f32", "bf16", "bf16", "fp8"])
    lo, hi, cap = {"f64": (128, 8192, 1.0e12), "f32": (128, 16384, 1.0e12), "bf16": (256, 16384, 6.0e12),
                   "fp8": (256, 16384, 6.0e12)}[dtype]
    vec = 16 // SIZE[dtype]
    while True:
        m, n, k = (_log(rng, lo, hi) for _ in range(3))
        # inner sizes: whole 128-byte slabs or only whole 16-byte vectors
        unit = 128 // SIZE[dtype] if rng.random() < 0.5 else vec
        k = max(unit, k // unit * unit)
        b = 1 if rng.random() < 0.65 else rng.choice([16, 32, 64, 128] if dtype in ("f64", "f32") else [16, 32])
        if b > 1:
            m, n = max(2, m // b) * b, max(2, n // b) * b
        if 2.0 * m * n * k <= cap:
            break
    return _step(None, dtype, m, n, k, b, b, fused=b == 1 and rng.random() < 0.3, rebuild=b > 1,
                 correct=b == 1 and dtype == "f64" and rng.random() < 0.5)


def draw(rng):
    x = rng.random()
    if x < 0.68:
        return _draw_step(rng)
    if x < 0.76:
        b, panels = rng.choice([64, 128, 256]), rng.choice([2, 4, 8])
        m, n = (b * rng.randint(2, 3072 // b) for _ in range(2))
        return _panels(None, m, n, 16 * panels * rng.randint(4, 2048 // (16 * panels)), b, panels)
    if x < 0.84:
        b = rng.choice([64, 128, 256, 512])
        m, n = (b * rng.randint(4, 5120 // b) for _ in range(2))
        dtype = rng.choice(["f64", "f64", "f32"])
        # binary32: one lost block (its rebuild divides by one weight; a solve would magnify the roundings)
        return _weighted(None, dtype, m, n, 4 * _log(rng, 64, 1024), b, 1 if dtype == "f32" else rng.choice([1, 2, 3]))
    if x < 0.90:
        b = rng.choice([128, 256, 512])
        return {"kind": "matvec", "m": b * rng.randint(4, 16384 // b), "k": 2 * _log(rng, 512, 8192), "b": b,
                "f": rng.choice([1, 2])}
    return _batch(None, _log(rng, 4, 512), 32 * _log(rng, 8, 64), rng.choice([1, 32]), rng.randrange(1 << 30))


# ---------------------------------------------------------------- inputs
def _gen(seed, device):
    return torch.Generator(device=device).manual_seed(seed)


def _uniform(gen, rows, cols, dtype):
    return torch.empty(rows, cols, dtype=dtype, device=gen.device).uniform_(-1, 1, generator=gen)


def _step_inputs(case, seed):
    """A (m x k) and B^T (n x k): binary64 for f64, else binary32."""
    gen = _gen(seed, "cuda")
    dt = torch.float64 if case.get("dtype", "f64") == "f64" else torch.float32
    return _uniform(gen, case["m"], case["k"], dt), _uniform(gen, case.get("n", 1), case["k"], dt)


def _lost_block(case):
    """A data block of the block grid, as (i0, j0, h, w)."""
    br, bc = case.get("br", case.get("b")), case.get("bc", case.get("b"))
    return ((case["m"] // br) // 2 * br, (case["n"] // bc) // 3 * bc, br, bc)


def _weights(seed, f, groups):
    return 0.5 + np.random.RandomState(seed).random_sample((f, groups))


def _batch_layout(case):
    """Shapes of the batch and the offset of every problem's A, B^T and C_f in
    flat buffers (C rows padded to 16 bytes, every matrix on a 256-byte boundary)."""
    rs = np.random.RandomState(case["shapes_seed"] % (1 << 31))
    span = (case["hi"] - case["lo"]) // case["step"] + 1
    shapes = (case["lo"] + case["step"] * rs.randint(0, span, (case["count"], 3))).tolist()
    up = lambda v: (v + 127) // 128 * 128  # noqa: E731
    at, off = [], [0, 0, 0]
    for m, n, k in shapes:
        ldc = (n + 1 + 3) // 4 * 4
        at.append((off[0], off[1], off[2], ldc))
        off = [off[0] + up(m * k), off[1] + up(n * k), off[2] + up((m + case["br"]) * ldc)]
    return shapes, at, off


def _batch_inputs(case, seed):
    shapes, at, (na, nb, nc) = _batch_layout(case)
    gen = _gen(seed, "cuda")
    return shapes, at, nc, _uniform(gen, 1, na, torch.float32)[0], _uniform(gen, 1, nb, torch.float32)[0]


# ---------------------------------------------------------------- prepare
def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def _prepare_step(case, seed):
    dt = case["dtype"]
    P = abft.Protected(DTYPES[dt], case["m"], case["n"], case["k"], case["br"], case["bc"])
    A, Bt = _step_inputs(case, seed)
    st = {"case": case, "P": P}
    if dt in ("f64", "f32"):
        P.A[:case["m"]].copy_(A)
        P.Bt[:case["n"]].copy_(Bt)
    else:
        st["A32"], st["B32"] = A, Bt
    if case["rebuild"]:
        st["lost"] = _lost_block(case)
    if case["correct"]:
        st["loc"] = abft.abft_location(abft.ABFT_CLS_DATA, abft.ABFT_DIR_COL, case["m"] // 3, case["n"] // 2)
    return st


def _prepare_panels(case, seed):
    P = abft.Protected(abft.ABFT_F64, case["m"], case["n"], case["k"], case["b"], case["b"])
    A, Bt = _step_inputs(case, seed)
    P.A[:case["m"]].copy_(A)
    P.Bt[:case["n"]].copy_(Bt)
    return {"case": case, "P": P, "lost": _lost_block(case)}


def _prepare_weighted(case, seed):
    m, n, k, b, f = (case[q] for q in ("m", "n", "k", "b", "f"))
    P = abft.WProtected(m, n, k, b, b, _weights(seed, f, m // b), _weights(seed + 1, f, n // b),
                        dtype=DTYPES[case["dtype"]])
    A, Bt = _step_inputs(case, seed)
    P.A[:m].copy_(A)
    P.Bt[:n].copy_(Bt)
    lost = [(m // b) // 2 + q for q in range(f)]
    j0 = (n // b) // 3 * b
    return {"case": case, "P": P, "lost": lost, "j0": j0, "known": [(g * b, j0, b, b) for g in lost]}


def _prepare_matvec(case, seed):
    m, k, b, f = (case[q] for q in ("m", "k", "b", "f"))
    P = abft.WProtected(m, 1, k, b, 1, _weights(seed, f, m // b), [[1.0]])
    A, x = _step_inputs(case, seed)
    P.A[:m].copy_(A)
    P.Bt[:1].copy_(x)
    return {"case": case, "P": P}


def _prepare_batch(case, seed):
    shapes, at, nc, A32, B32 = _batch_inputs(case, seed)
    A, B = (torch.zeros_like(x, dtype=torch.bfloat16) for x in (A32, B32))
    C = torch.zeros(nc, dtype=torch.float32, device="cuda")
    probs, items = [], []
    for (m, n, k), (a, b, c, ldc) in zip(shapes, at):
        probs.append(abft.problem(abft.ABFT_BF16, m, n, k, case["br"], 1, ldc=ldc, lam=20.0))
        items.append(abft.abft_batch_item(A32.data_ptr() + 4 * a, B32.data_ptr() + 4 * b, A.data_ptr() + 2 * a,
                                          B.data_ptr() + 2 * b, C.data_ptr() + 4 * c))
    bws = torch.zeros(abft.batch_workspace_size(probs), dtype=torch.uint8, device="cuda")
    plan = abft.batch_setup(probs, items, bws)
    abft.batch_quantize_encode(plan)
    tile = abft.batch_choose(plan)[1]
    rep = torch.empty(len(probs) * abft.C.sizeof(abft.abft_report), dtype=torch.uint8, pin_memory=True)
    return {"case": case, "plan": plan, "tile": tile, "A32": A32, "B32": B32, "A": A, "B": B, "C": C, "bws": bws,
            "rep": rep}


_PREPARE = {"step": _prepare_step, "panels": _prepare_panels, "weighted": _prepare_weighted,
            "matvec": _prepare_matvec, "batch": _prepare_batch}


# ---------------------------------------------------------------- run
def run(state):
    return _RUN[state["case"]["kind"]](state)


def _counts(rep):
    return [rep.n_flag_c, rep.n_flag_r, rep.n_excl_c, rep.n_excl_r, rep.n_nonfinite, rep.status]


def _wcounts(rep):
    return [rep.n_fail_c, rep.n_fail_r, rep.n_excl_c, rep.n_excl_r]


def _run_step(st):
    case, P = st["case"], st["P"]
    m, n = case["m"], case["n"]
    lowp = "A32" in st
    if lowp:
        abft.quantize_encode(P.p, st["A32"], st["B32"], P.A, P.Bt, P.ws)
    else:
        P.encode()
    P.gemm(abft.ABFT_FUSED if case["fused"] else 0)
    known = [st["lost"]] if case["rebuild"] else None
    rep = P.verify_fused() if case["fused"] else P.verify(known)
    out = {"report": _counts(rep), "class": abft.classify(P.p, rep, known).cls}
    if case["rebuild"]:
        abft.recover_block(P.p, P.C, st["lost"])
        out["again"] = _counts(P.verify())
    if case["correct"]:
        abft.correct(P.p, P.C, st["loc"])
        out["again"] = _counts(P.verify())
    # what the pass wrote: the quantized operands, or the operands' checksum rows and columns
    out.update({"A": P.A, "B": P.Bt} if lowp else {"A_rows": P.A[m:], "B_cols": P.Bt[n:]})
    out["C"] = P.C
    return out


def _run_panels(st):
    case, P = st["case"], st["P"]
    k, panels = case["k"], case["panels"]
    P.encode()
    for q in range(panels):
        if q == panels // 2:
            rep = P.verify([st["lost"]])
            abft.recover_block(P.p, P.C, st["lost"])
        abft.gemm_panel(P.p, P.A, P.Bt, P.C, q * k // panels, (q + 1) * k // panels, abft.ABFT_ACCUMULATE if q else 0)
    again = P.verify()
    return {"report": _counts(rep), "again": _counts(again), "A_rows": P.A[case["m"]:], "B_cols": P.Bt[case["n"]:],
            "C": P.C}


def _run_weighted(st):
    case, P = st["case"], st["P"]
    P.encode()
    P.gemm()
    rep = P.verify(st["known"])
    abft.wrecover(P.p, P.C, abft.ABFT_DIR_COL, st["lost"], st["j0"], case["b"], P.ws)
    again = P.verify()
    return {"report": _wcounts(rep), "again": _wcounts(again), "A_rows": P.A[case["m"]:], "B_cols": P.Bt[case["n"]:],
            "C": P.C}


def _run_matvec(st):
    case, P = st["case"], st["P"]
    P.encode()
    P.gemm()
    rep = P.verify()
    return {"report": _wcounts(rep), "A_rows": P.A[case["m"]:], "B_cols": P.Bt[1:], "C": P.C}


def _run_batch(st):
    plan = st["plan"]
    abft.batch_quantize_encode(plan)
    abft.batch_gemm(plan, st["tile"])
    abft.batch_verify(plan)
    abft.batch_reports(plan, st["rep"])
    torch.cuda.current_stream().synchronize()
    words = st["rep"].numpy().view(np.int64).reshape(st["case"]["count"], -1)
    return {"reports": words[:, :REPORT_WORDS].copy(), "A": st["A"], "B": st["B"], "C": st["C"]}


_RUN = {"step": _run_step, "panels": _run_panels, "weighted": _run_weighted, "matvec": _run_matvec,
        "batch": _run_batch}


# ---------------------------------------------------------------- exact
def exact(case, seed):
    return _EXACT[case["kind"]](case, seed)


def _fp8_values(X):
    """E4M3 values after the per-tensor power-of-two scale, scaled back: the
    largest e with max|X| 2^e <= 448, x 2^e rounded to nearest even."""
    amax = float(X.abs().max().double())
    e = 0
    if amax > 0:
        e = int(np.floor(np.log2(448.0 / amax)))
        while amax * 2.0 ** (e + 1) <= 448.0:
            e += 1
        while amax * 2.0 ** e > 448.0:
            e -= 1
    return (X.double() * 2.0 ** e).float().to(torch.float8_e4m3fn).double() * 2.0 ** -e


def _block_sums(X, b):
    return torch.cat([X, X.view(X.shape[0] // b, b, X.shape[1]).sum(0)])


def _exact_step(case, seed):
    dt = case.get("dtype", "f64")
    br, bc = case.get("br", case.get("b")), case.get("bc", case.get("b"))
    A, Bt = _step_inputs(case, seed)
    lowp = dt in ("bf16", "fp8")
    if dt == "bf16":
        A, Bt = A.bfloat16(), Bt.bfloat16()
    elif dt == "fp8":
        A, Bt = _fp8_values(A), _fp8_values(Bt)
    A, Bt = _block_sums(A.double(), br), _block_sums(Bt.double(), bc)
    out = {"report": None, "class": None, "again": None, "C": A @ Bt.t()}
    if dt == "bf16":
        out.update({"A": A[:case["m"]], "B": Bt[:case["n"]]})
    elif not lowp:
        out.update({"A_rows": A[case["m"]:], "B_cols": Bt[case["n"]:]})
    return out


def _weighted_sums(X, b, w):
    blocks = X.view(X.shape[0] // b, b * X.shape[1])
    return torch.cat([X, (torch.from_numpy(w).to(X.device) @ blocks).view(-1, X.shape[1])])


def _exact_weighted(case, seed):
    m, n, b, f = case["m"], case.get("n", 1), case["b"], case["f"]
    A, Bt = (X.double() for X in _step_inputs(case, seed))
    A = _weighted_sums(A, b, _weights(seed, f, m // b))
    Bt = torch.cat([Bt, Bt]) if case["kind"] == "matvec" else _weighted_sums(Bt, b, _weights(seed + 1, f, n // b))
    return {"report": None, "again": None, "A_rows": A[m:], "B_cols": Bt[n:], "C": A @ Bt.t()}


def _exact_batch(case, seed):
    shapes, at, nc, A32, B32 = _batch_inputs(case, seed)
    A, B = A32.bfloat16(), B32.bfloat16()
    C = torch.zeros(nc, dtype=torch.float64, device="cuda")
    for (m, n, k), (a, b, c, ldc) in zip(shapes, at):
        X = _block_sums(A[a:a + m * k].view(m, k).double(), case["br"])
        Y = _block_sums(B[b:b + n * k].view(n, k).double(), 1)
        C[c:c + X.shape[0] * ldc].view(-1, ldc)[:, :n + 1] = X @ Y.t()
    # elements of the flat operands between two problems are never written
    used = [torch.zeros_like(x, dtype=torch.bool) for x in (A, B)]
    for (m, n, k), (a, b, _, _) in zip(shapes, at):
        used[0][a:a + m * k] = True
        used[1][b:b + n * k] = True
    return {"reports": None, "A": A.double() * used[0], "B": B.double() * used[1], "C": C}


_EXACT = {"step": _exact_step, "panels": _exact_step, "weighted": _exact_weighted, "matvec": _exact_weighted,
          "batch": _exact_batch}


# ---------------------------------------------------------------- work
def _one(m, n, k, M, N, in_size, stored_size, c_size):
    """Operands read once as they come in (stored_size bytes more per element
    where they are quantized), checksum rows and C_f written once, C_f read
    once by the verification; the products of the encoded operands."""
    return {"bytes": (m + n) * k * (in_size + stored_size) + (M - m + N - n) * k * max(in_size, 4) + 2 * M * N * c_size,
            "flops": 2.0 * M * N * k}


def work(case):
    kind = case["kind"]
    if kind == "batch":
        shapes, _, _ = _batch_layout(case)
        each = [_one(m, n, k, m + case["br"], n + 1, 4, 2, 4) for m, n, k in shapes]
        return {q: float(sum(w[q] for w in each)) for q in ("bytes", "flops")}
    m, n, k, dt = case["m"], case.get("n", 1), case["k"], case.get("dtype", "f64")
    c_size = 8 if dt == "f64" else 4
    if kind in ("weighted", "matvec"):
        fc = 1 if kind == "matvec" else case["f"]
        b = 1 if kind == "matvec" else case["b"]
        return _one(m, n, k, m + case["f"] * case["b"], n + fc * b, SIZE[dt], 0, c_size)
    br, bc = case.get("br", case.get("b")), case.get("bc", case.get("b"))
    lowp = dt in ("bf16", "fp8")
    return _one(m, n, k, m + br, n + bc, 4 if lowp else SIZE[dt], SIZE[dt] if lowp else 0, c_size)
