"""GPU test of the statistical thresholds at operand scales far from one: A
scaled by 2^70 and B by 2^-70, and the reverse, is a product of ordinary
magnitude, but the weights of the thin-block statistics (sums of squares of
the other operand) are near 2^140 and 2^-140, outside binary32's range.  The
thresholds of both directions must be the oracle's (a C_f of NaN fails every
relation, so each report lists 64 of each direction), a clean product must
verify, and a flipped element must be located -- also in a column where B
holds zeros, whose products with an overflowed weight would be NaN.

The sizes take every way the weighted row statistic is formed: k of whole and
of partial strips, several weight slabs with a short last one, few rows and
many, and B large enough for the serial passes.

Tolerance: the statistics are binary64 sums of at most k + G terms, so a
threshold carries a relative error of a few (k + G) 2^-53 < 1e-10."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_0806_3121_amd import abft, synth  # noqa: E402

pytestmark = pytest.mark.gpu

SEED = synth.BASE_SEED + 211
DT = {"f32": abft.ABFT_F32, "bf16": abft.ABFT_BF16}

CASES = [
    # dtype, m, n, k, br, bc
    ("f32", 130, 200, 256, 1, 1),       # whole strips
    ("f32", 200, 130, 260, 1, 1),       # partial strips
    ("f32", 96, 60, 8708, 1, 1),        # three weight slabs, the last one short
    ("f32", 60, 9001, 64, 1, 1),        # many rows, ragged
    ("bf16", 130, 200, 512, 1, 1),
    ("bf16", 200, 130, 520, 1, 1),
    ("bf16", 60, 96, 4616, 1, 1),
    ("bf16", 9004, 48, 136, 4, 1),      # weighted rows of A only
    ("bf16", 48, 9003, 136, 1, 3),      # weighted rows of B only
    ("bf16", 40, 3200, 8192, 1, 1),     # B beyond the serial passes' size
]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    abft.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("ea", [70, -70])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_thresholds_and_decisions_far_from_one(dev, orc, case, ea):
    dt, m, n, k, br, bc = case
    print(f"[case] statistics at scale 2^{ea} {case}", flush=True)
    A = np.ldexp(synth.uniform(SEED, synth.STREAM_A, m, k, np.float32), ea).astype(np.float32)
    Bt = np.ldexp(synth.uniform(SEED, synth.STREAM_B, n, k, np.float32), -ea).astype(np.float32)
    Bt[n // 2, ::3] = 0.0
    A[m // 2, ::5] = 0.0
    P = abft.Protected(DT[dt], m, n, k, br, bc, device=dev, lam=10.0, tau_mode=abft.ABFT_TAU_STAT)
    Ad, Btd = torch.from_numpy(A).to(dev), torch.from_numpy(Bt).to(dev)
    if dt == "f32":
        P.A[:m], P.Bt[:n] = Ad, Btd
        P.encode()
        T = float(k)
    else:
        abft.quantize_encode(P.p, Ad, Btd, P.A, P.Bt, P.ws)
        A, Bt = (orc.bf16_bits_to_f64(orc.to_bf16_bits(X)) for X in (A, Bt))
        T = k / 4.0
    Af, Bf = orc.encode(A.astype(np.float64), np.ascontiguousarray(Bt.T).astype(np.float64), br, bc, store_f32=True)
    P.gemm()
    clean = P.C.clone()
    rep = P.verify()
    assert rep.n_flag_c == 0 and rep.n_flag_r == 0, (rep.max_ratio_c, rep.max_ratio_r)
    assert 0 < rep.max_ratio_c < 1 and 0 < rep.max_ratio_r < 1
    i, j = m // 3, n // 2
    abft.inject_flip(P.p, P.C, i, j, 28)
    loc = abft.classify(P.p, P.verify())
    assert (loc.cls, loc.i, loc.j) == (abft.ABFT_CLS_DATA, i, j)
    abft.correct(P.p, P.C, loc)
    rep = P.verify()
    assert rep.n_flag_c == 0 and rep.n_flag_r == 0
    assert (P.C - clean).abs().max().item() <= 1e-4 * clean.abs().max().item()
    tc, tr = orc.tau_stat(Af, Bf, m, n, br, bc, T=T, s_store=2.0, lam=10.0)
    P.C.fill_(float("nan"))
    rep = P.verify()
    assert rep.n_flag_c == br * (n + bc) and rep.n_flag_r == (m + br) * bc
    for r, jj, _, tau in rep.flags_c():
        assert abs(tau - tc[r, jj]) <= 1e-10 * tc[r, jj], (r, jj, tau, tc[r, jj])
    for ii, c, _, tau in rep.flags_r():
        assert abs(tau - tr[ii, c]) <= 1e-10 * tr[ii, c], (ii, c, tau, tr[ii, c])


@pytest.mark.parametrize("ea", [70, -70])
def test_batched_thresholds_far_from_one(dev, orc, ea):
    """The same of the batched products: every threshold of every problem."""
    print(f"[case] batched statistics at scale 2^{ea}", flush=True)
    shapes = [(130, 96, 64, 1, 1), (96, 130, 520, 1, 1), (64, 60, 2048, 1, 1), (48, 40, 4616, 1, 1), (60, 64, 136, 4, 1),
              (64, 60, 136, 1, 4)]
    bt = abft.Batch(shapes, device=dev, lam=10.0)
    host = []
    for q, (m, n, k, _, _) in enumerate(shapes):
        A = np.ldexp(synth.uniform(SEED + q, synth.STREAM_A, m, k, np.float32), ea).astype(np.float32)
        Bt = np.ldexp(synth.uniform(SEED + q, synth.STREAM_B, n, k, np.float32), -ea).astype(np.float32)
        Bt[n // 2, ::3] = 0.0
        A[m // 2, ::5] = 0.0
        bt.A32[q].copy_(torch.from_numpy(A))
        bt.Bt32[q].copy_(torch.from_numpy(Bt))
        host.append(tuple(orc.bf16_bits_to_f64(orc.to_bf16_bits(X)).astype(np.float64) for X in (A, Bt)))
    abft.batch_quantize_encode(bt.plan)
    abft.batch_gemm(bt.plan)
    abft.batch_verify(bt.plan)
    assert bt.fetch_reports() == []
    for q, (m, n, k, br, bc) in enumerate(shapes):
        A, Bt = host[q]
        Af, Bf = orc.encode(A, np.ascontiguousarray(Bt.T), br, bc, store_f32=True)
        Cf = bt.C[q].cpu().numpy().astype(np.float64)
        tc, tr = orc.tau_stat(Af, Bf, m, n, br, bc, T=k / 4.0, s_store=2.0, lam=10.0, Cf=Cf, T_c=k / 4.0)
        tau_c = torch.zeros(br, n + bc, dtype=torch.float64, device=dev)
        tau_r = torch.zeros(m + br, bc, dtype=torch.float64, device=dev)
        abft.batch_thresholds(bt.plan, q, tau_c, tau_r)
        for got, want in ((tau_c.cpu().numpy(), tc), (tau_r.cpu().numpy(), tr)):
            assert np.all(np.abs(got - want) <= 1e-10 * want), (q, np.max(np.abs(got - want) / want))
