"""GPU test of the report's maxima beside excluded relations: with a block known
lost, the largest ratio of each direction is that of the relations still judged,
and it reaches the report from blocks that count exclusions and from blocks that
do not, in every verification kernel.

Two elements outside the lost block's rows and columns are wrong by amounts three
apart, a third inside its rows: every failing relation is listed, and the maximum
is the largest |d| / tau of the list, the same division of the same two numbers:
no tolerance."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_0806_3121_amd import abft, synth  # noqa: E402

pytestmark = pytest.mark.gpu

SEED = synth.BASE_SEED + 239
DT = {"f64": abft.ABFT_F64, "f32": abft.ABFT_F32, "bf16": abft.ABFT_BF16, "fp8": abft.ABFT_FP8_E4M3}

CASES = [
    # dtype, m, n, k, br, bc
    ("f64", 1024, 1024, 64, 128, 128),      # one pass, wide blocks
    ("f64", 700, 600, 64, 50, 75),          # a residue per thread
    ("f64", 2000, 300, 32, 4, 4),           # a wave per row
    ("f32", 800, 1200, 64, 100, 120),       # several residues per load
    ("f32", 500, 400, 64, 1, 1),            # tile partial sums
    ("bf16", 500, 400, 64, 1, 1),
    ("fp8", 640, 320, 64, 8, 16),
]


@pytest.mark.parametrize("big_first", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_maximum_beside_excluded_relations(case, big_first):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dt, m, n, k, br, bc = case
    print(f"[case] maximum beside exclusions {case} {big_first}", flush=True)
    lowp = dt in ("bf16", "fp8")
    npd = np.float64 if dt == "f64" else np.float32
    P = abft.Protected(DT[dt], m, n, k, br, bc, lam=10.0, tau_mode=abft.ABFT_TAU_DET)
    A = torch.from_numpy(synth.uniform(SEED, synth.STREAM_A, m, k, npd)).cuda()
    Bt = torch.from_numpy(synth.uniform(SEED, synth.STREAM_B, n, k, npd)).cuda()
    if lowp:
        abft.quantize_encode(P.p, A, Bt, P.A, P.Bt, P.ws)
    else:
        P.A[:m], P.Bt[:n] = A, Bt
        P.encode()
    P.gemm()
    rect = (br * 2, bc * 2, br, bc)
    abft.inject_erase(P.p, P.C, rect, True)
    amounts = (3000.0, 1000.0) if big_first else (1000.0, 3000.0)
    P.C[0, 0] += amounts[0]
    P.C[m - 1, n - 1] += amounts[1]
    P.C[2 * br, 0] += 9000.0            # its row relations of the lost block's columns are excluded
    rep = P.verify(known=[rect])
    assert rep.n_excl_c == br * bc and rep.n_excl_r == br * bc
    for nf, flags, top in ((rep.n_flag_c, rep.flag_c, rep.max_ratio_c), (rep.n_flag_r, rep.flag_r, rep.max_ratio_r)):
        assert 2 <= nf <= 4
        assert top == max(abs(flags[q].d) / flags[q].tau for q in range(nf))
