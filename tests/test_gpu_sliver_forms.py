"""GPU test of the carried blocks' forms: every count of checksum rows a launch
takes (one to eight, and a remainder), the corner entry by entry and by tiles
(ragged in both directions), several operand rows per wave with k of one short
chunk and of more, in every element type.

The operands hold integers in [-2, 2], so checksum sums, products and the
binary64 sums of the carried blocks are exact and below 2^24: C_f must equal
the integer product of the encoded operands, no tolerance."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_0806_3121_amd import abft, synth  # noqa: E402

pytestmark = pytest.mark.gpu

SEED = synth.BASE_SEED + 227
DT = {"f64": abft.ABFT_F64, "f32": abft.ABFT_F32, "bf16": abft.ABFT_BF16, "fp8": abft.ABFT_FP8_E4M3}

CASES = [(dt, 3 * b, 2 * c, k, b, c) for dt in ("f64", "f32", "bf16", "fp8")
         for b, c, k in ((1, 1, 16), (2, 3, 528), (3, 2, 272), (4, 8, 1040), (5, 7, 48), (8, 6, 2064))]
CASES += [("bf16", 18, 34, 24, 9, 17), ("fp8", 34, 18, 1104, 17, 9)]                       # more than one group of eight
CASES += [("bf16", 262, 260, 264, 131, 130), ("fp8", 130, 264, 48, 130, 132),              # corner by tiles
          ("bf16", 6, 5500, 16, 3, 5500), ("fp8", 128, 128, 2064, 128, 128)]
CASES += [("f64", 16400, 6, k, 2, 1) for k in (2, 128, 130, 256, 258)]                     # several rows per wave
CASES += [("f32", 16390, 4, 20, 1, 2), ("bf16", 16389, 5, 8, 1, 1), ("fp8", 16400, 6, 32, 2, 2)]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    abft.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_carried_blocks_are_exact(dev, case):
    dt, m, n, k, br, bc = case
    print(f"[case] carried blocks {case}", flush=True)
    lowp = dt in ("bf16", "fp8")
    A = synth.uniform_ints(SEED, synth.STREAM_A, m, k, -2, 2).astype(np.float64)
    Bt = synth.uniform_ints(SEED, synth.STREAM_B, n, k, -2, 2).astype(np.float64)
    P = abft.Protected(DT[dt], m, n, k, br, bc, device=dev, lam=10.0)
    assert ("k_corner" in abft.describe_gemm(P.p)) == (lowp and br * bc >= 128 * 128)
    Ad, Btd = (torch.from_numpy(X.astype(np.float64 if dt == "f64" else np.float32)).to(dev) for X in (A, Bt))
    if lowp:
        abft.quantize_encode(P.p, Ad, Btd, P.A, P.Bt, P.ws)
    else:
        P.A[:m], P.Bt[:n] = Ad, Btd
        P.encode()
    P.C.fill_(float("nan"))
    P.gemm()
    Af = np.vstack([A, A.reshape(m // br, br, k).sum(axis=0)])
    Bf = np.vstack([Bt, Bt.reshape(n // bc, bc, k).sum(axis=0)])
    assert np.array_equal(P.C.cpu().numpy().astype(np.float64), Af @ Bf.T)
    rep = P.verify()
    assert rep.n_flag_c == 0 and rep.n_flag_r == 0


@pytest.mark.parametrize("dt,m,k", [("f64", 16400, 100), ("f64", 16400, 300), ("f32", 17, 64)])
def test_accumulating_panels_add_to_the_carried_blocks(dev, dt, m, k):
    print(f"[case] carried blocks accumulated {dt} m={m} k={k}", flush=True)
    n = 5
    A = synth.uniform_ints(SEED, synth.STREAM_A, m, k, -2, 2).astype(np.float64)
    Bt = synth.uniform_ints(SEED, synth.STREAM_B, n, k, -2, 2).astype(np.float64)
    P = abft.Protected(DT[dt], m, n, k, 1, 1, device=dev, lam=10.0)
    P.A[:m], P.Bt[:n] = torch.from_numpy(A).to(dev), torch.from_numpy(Bt).to(dev)
    P.encode()
    for q in range(2):
        abft.gemm_panel(P.p, P.A, P.Bt, P.C, q * k // 2 // 4 * 4, k if q else k // 2 // 4 * 4, abft.ABFT_ACCUMULATE if q else 0)
    Af, Bf = np.vstack([A, A.sum(axis=0)]), np.vstack([Bt, Bt.sum(axis=0)])
    assert np.array_equal(P.C.cpu().numpy().astype(np.float64), Af @ Bf.T)
