"""The bfloat16 / FP8 tiles of the half-slab ring against exact integer
products: every tile with k a multiple of the 64-byte half, one vector over,
and one vector short of it, fewer halves than the ring holds, and ragged m and
n so every tile has partial edge tiles.  Each case names the tile that runs.

Integer operands in [-4, 4] are exact in both element types and every partial
sum is an integer of magnitude at most 16 k < 2^24 (times a power of two in the
FP8 domain), so the product must be equal whatever the summation order: no
tolerance.  The fused product must give the same bits on its own tile."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_0806_3121_amd import abft, synth  # noqa: E402

pytestmark = pytest.mark.gpu

SEED = synth.BASE_SEED + 157
DT = {"bf16": abft.ABFT_BF16, "fp8": abft.ABFT_FP8_E4M3}

CASES = [
    ("bf16", 300, 260, 512, "64x64"),
    ("bf16", 65, 127, 520, "64x64"),
    ("bf16", 900, 765, 1048, "64x64"),
    ("bf16", 260, 300, 8, "128x128"),        # one vector of k
    ("bf16", 260, 300, 104, "128x128"),      # four halves, the last one short
    ("bf16", 1487, 2040, 200, "128x128"),
    ("bf16", 440, 11551, 232, "256x128"),
    ("bf16", 3000, 5003, 264, "256x256"),
    ("bf16", 3000, 5003, 24, "256x256"),
    ("bf16", 3000, 5003, 96, "256x256"),
    ("fp8", 300, 260, 1024, "64x64"),
    ("fp8", 65, 127, 1040, "64x64"),
    ("fp8", 260, 300, 16, "128x128"),
    ("fp8", 260, 300, 208, "128x128"),
    ("fp8", 1487, 2040, 464, "128x128"),
    ("fp8", 440, 11551, 464, "256x128"),
    ("fp8", 3000, 5003, 528, "256x256"),
    ("fp8", 3000, 5003, 192, "256x256"),
]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    abft.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_ring_tile_is_exact(dev, case):
    dt, m, n, k, tile = case
    print(f"[case] ring tile {case}", flush=True)
    A = synth.uniform_ints(SEED, synth.STREAM_A, m, k, -4, 4)
    B = synth.uniform_ints(SEED, synth.STREAM_B, k, n, -4, 4)
    P = abft.Protected(DT[dt], m, n, k, 1, 1, device=dev, tau_mode=abft.ABFT_TAU_STAT, lam=10.0)
    desc = abft.describe_gemm(P.p, abft.ABFT_PLAIN)
    assert desc.startswith(f"k_gemm_lowp {dt} {tile} on {m}x{n} k={k}"), desc
    abft.quantize(P.p, 0, torch.from_numpy(A.astype(np.float32)).to(dev), P.A, P.ws)
    abft.quantize(P.p, 1, torch.from_numpy(np.ascontiguousarray(B.T).astype(np.float32)).to(dev), P.Bt, P.ws)
    P.encode()
    want = (A.astype(np.float64) @ B.astype(np.float64)).astype(np.float32)
    for fused in (False, True):
        P.C.fill_(float("nan"))
        abft.gemm(P.p, P.A, P.Bt, P.C, P.ws, abft.ABFT_FUSED if fused else 0)
        assert np.array_equal(P.C[:m, :n].cpu().numpy(), want)
        rep = P.verify()
        assert rep.n_flag_c == 0 and rep.n_flag_r == 0


@pytest.mark.parametrize("dt,m,n,k", [("bf16", 300, 260, 520), ("bf16", 440, 11551, 232), ("bf16", 3000, 5003, 264)])
def test_infinities_stay_in_their_rows(dev, dt, m, n, k):
    """An infinite operand entry at the end of k reaches its own row (or
    column) only: the masked part of the last half multiplies nothing."""
    print(f"[case] infinity at the end of k {dt} {m}x{n}x{k}", flush=True)
    A = torch.ones(m, k, dtype=torch.bfloat16, device=dev)
    Bt = torch.ones(n, k, dtype=torch.bfloat16, device=dev)
    A[7, k - 1] = float("inf")
    Bt[n - 2, k - 2] = float("inf")
    p = abft.problem(DT[dt], m, n, k, 1, 1, ldc=n)
    C = torch.zeros(m, n, dtype=torch.float32, device=dev)
    abft.gemm(p, A, Bt, C, None, abft.ABFT_PLAIN)
    inf = torch.isinf(C)
    want = torch.zeros_like(inf)
    want[7, :] = True
    want[:, n - 2] = True
    assert torch.equal(inf, want) and not torch.isnan(C).any()
    assert (C[~want] == k).all()
