"""GPU test of the encode pass's split over blocks: 64- and 16-lane strips
with ragged last lanes, whole residues per lane and partitioned sums, both
operands in one launch and one after the other, row statistics taken in the
pass and in a pass of their own.  The checksum rows and the thresholds built
from the statistics are compared with the oracle's: a C_f of NaN fails every
relation, so each report lists 64 thresholds of each direction.

Tolerances: checksum rows are binary64 sums of G terms, rounded once (at most
G 2^-53 times the sum of magnitudes, which is below G here); a det threshold
carries relative errors of a few (k + G) 2^-53, a statistical one the
rounding of its weights to binary32 as well (2^-24)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_0806_3121_amd import abft, synth  # noqa: E402

pytestmark = pytest.mark.gpu

SEED = synth.BASE_SEED + 131
DT = {"f64": abft.ABFT_F64, "f32": abft.ABFT_F32, "bf16": abft.ABFT_BF16, "fp8": abft.ABFT_FP8_E4M3}

CASES = [
    ("f64", 150, 70, 258, 1, 1),        # 129 vectors: 16-lane strips, one lane in the last
    ("f64", 96, 128, 128, 32, 64),      # few groups: whole residues per lane, 64-lane strips
    ("f64", 1400, 34, 1282, 2, 1),      # 641 vectors: 64-lane strips, one lane in the last; partitioned, 2 residues
    ("f64", 51, 2, 2, 3, 2),            # the smallest inner size; more row lanes than residues
    ("f32", 513, 700, 516, 1, 1),
    ("f32", 130, 256, 260, 1, 4),       # weighted statistic on one side only
    ("bf16", 300, 260, 1032, 1, 1),
    ("bf16", 64, 3200, 8192, 1, 1),     # B large enough for the serial passes
    ("fp8", 130, 200, 1040, 1, 1),
    ("fp8", 130, 300, 528, 13, 1),
]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    abft.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_checksums_and_thresholds_match_oracle(dev, orc, case):
    dt, m, n, k, br, bc = case
    print(f"[case] encode split {case}", flush=True)
    np_dt = np.float64 if dt == "f64" else np.float32
    A = synth.uniform(SEED, synth.STREAM_A, m, k, np_dt)
    Bt = synth.uniform(SEED, synth.STREAM_B, n, k, np_dt)
    stat = dt != "f64"
    P = abft.Protected(DT[dt], m, n, k, br, bc, device=dev, lam=10.0,
                       tau_mode=abft.ABFT_TAU_STAT if stat else abft.ABFT_TAU_DET)
    Ad, Btd = torch.from_numpy(A).to(dev), torch.from_numpy(Bt).to(dev)
    sc = 1.0
    if dt in ("f64", "f32"):
        P.A[:m], P.Bt[:n] = Ad, Btd
        P.encode()
    else:
        abft.quantize_encode(P.p, Ad, Btd, P.A, P.Bt, P.ws)
        if dt == "bf16":
            A, Bt = (orc.bf16_bits_to_f64(orc.to_bf16_bits(X)) for X in (A, Bt))
        else:
            ea, eb = orc.e4m3_scale_exp(A), orc.e4m3_scale_exp(Bt)
            A, Bt = (orc.e4m3_values(orc.to_e4m3_codes(np.ldexp(X, e))) for X, e in ((A, ea), (Bt, eb)))
            sc = 2.0 ** -(ea + eb)
    Af, Bf = orc.encode(A.astype(np.float64), np.ascontiguousarray(Bt.T).astype(np.float64), br, bc, store_f32=stat)
    if dt in ("f64", "f32"):
        u = 2.0 ** -53 if dt == "f64" else 2.0 ** -24    # binary32: a tie may round the other way
        assert np.abs(P.A[m:].cpu().numpy() - Af[m:]).max() <= (m / br) ** 2 * 2.0 ** -53 + stat * 2 * u * m / br
        assert np.abs(P.Bt[n:].cpu().numpy() - Bf[:, n:].T).max() <= (n / bc) ** 2 * 2.0 ** -53 + stat * 2 * u * n / bc
    if stat:
        s_store = 2.0 + (2.0 ** 18 if dt == "fp8" else 0.0)
        tc, tr = orc.tau_stat(Af, Bf, m, n, br, bc, T=k / 4.0 if dt in ("bf16", "fp8") else float(k),
                              s_store=s_store, lam=10.0)
    else:
        tc, tr = orc.tau_det(Af, Bf, m, n, br, bc)
    P.C.fill_(float("nan"))
    rep = P.verify()
    assert rep.n_flag_c == br * (n + bc) and rep.n_flag_r == (m + br) * bc
    tol = 1e-6 if stat else 1e-10
    for r, j, _, tau in rep.flags_c():
        assert abs(tau - sc * tc[r, j]) <= tol * sc * tc[r, j], (r, j, tau, sc * tc[r, j])
    for i, c, _, tau in rep.flags_r():
        assert abs(tau - sc * tr[i, c]) <= tol * sc * tr[i, c], (i, c, tau, sc * tr[i, c])
