"""The bfloat16 / FP8 ring by slabs against exact integer products: every tile
and ring depth with one to six slabs of k, the last one whole, one vector long
and one vector short, rows off 128-byte lines with NaN beside them, and ragged m
and n; and the fused epilogue of every tile that has one, judged through its own
partial sums, with an accumulator flipped in the last tile.

Integer operands in [-4, 4] are exact in both element types and every partial
sum is an integer of magnitude at most 16 k < 2^24, so the product must be equal
whatever the summation order: no tolerance."""
import pytest

torch = pytest.importorskip("torch")

from paper_0806_3121_amd import abft, synth  # noqa: E402

pytestmark = pytest.mark.gpu

SEED = synth.BASE_SEED + 229
DT = {"bf16": abft.ABFT_BF16, "fp8": abft.ABFT_FP8_E4M3}

# m, n, tile, slabs of k for which the tile is picked
SHAPES = [
    (5000, 61, "64x64", range(1, 7)),        # products no wider than the tile, deep ring
    (33000, 20, "64x64", range(1, 7)),       # more tiles than the deep ring holds at once
    (300, 259, "64x64", (9, 10)),
    (259, 300, "128x128", range(1, 7)),      # deep ring
    (384, 19999, "128x128", range(1, 7)),    # two slabs, two blocks per CU
    (440, 11551, "256x128", range(1, 7)),    # three slabs
    (3000, 5003, "256x256", range(1, 7)),
]
CASES = [(dt, m, n, tile, s) for dt in ("bf16", "fp8") for m, n, tile, slabs in SHAPES for s in slabs]
CASES += [("fp8", m, n, "64x64", s) for m, n in ((33000, 190), (66, 3001)) for s in range(1, 4)]    # short k, narrow


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    abft.lib()
    return torch.device("cuda:0")


def operands(dev, dt, rows, k, seed, pad):
    """(rows, k) integers in [-4, 4] as binary64 and as stored with rows of k + pad elements, NaN in the padding."""
    gen = torch.Generator(device=dev).manual_seed(seed)
    X = torch.randint(-4, 5, (rows, k), device=dev, generator=gen)
    if dt == "bf16":
        S = torch.full((rows, k + pad), float("nan"), dtype=torch.bfloat16, device=dev)
        S[:, :k] = X.to(torch.bfloat16)
    else:
        codes = torch.tensor([0xC8, 0xC4, 0xC0, 0xB8, 0x00, 0x38, 0x40, 0x44, 0x48], dtype=torch.uint8, device=dev)
        S = torch.full((rows, k + pad), 0x7F, dtype=torch.uint8, device=dev)
        S[:, :k] = codes[X + 4]
    return X.double(), S


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_every_slab_count_is_exact(dev, case):
    dt, m, n, tile, slabs = case
    slab, vec = (64, 8) if dt == "bf16" else (128, 16)
    ks = sorted({k for k in ((slabs - 1) * slab + vec, slabs * slab - vec, slabs * slab) if k >= vec})
    for k in ks:
        pad = vec if k % slab == 0 else (0 if k % (2 * vec) else vec)
        print(f"[case] ring by slabs {case} k={k} pad={pad}", flush=True)
        p = abft.problem(DT[dt], m, n, k, 1, 1, lda=k + pad, ldb=k + pad, ldc=n)
        desc = abft.describe_gemm(p, abft.ABFT_PLAIN)
        if desc.startswith("k_gemm_lowp2"):
            continue                                   # whole slabs of 256 x 256: the other kernel's
        assert desc.startswith(f"k_gemm_lowp {dt} {tile} on {m}x{n} k={k}"), desc
        A, As = operands(dev, dt, m, k, SEED % 9973 + k, pad)
        B, Bs = operands(dev, dt, n, k, SEED % 9973 + k + 1, pad)
        ws = torch.zeros(abft.workspace_size(p), dtype=torch.uint8, device=dev)    # FP8 scale exponents 0
        C = torch.full((m, n), float("nan"), dtype=torch.float32, device=dev)
        abft.gemm(p, As, Bs, C, ws, abft.ABFT_PLAIN)
        assert torch.equal(C, (A @ B.t()).float())


@pytest.mark.parametrize("dt", ["bf16", "fp8"])
@pytest.mark.parametrize("m,n,tile", [(259, 300, "128x128"), (384, 19999, "128x128"), (440, 11551, "256x128"),
                                      (3000, 5003, "256x256")])
@pytest.mark.parametrize("slabs", [1, 3])
def test_fused_sums_of_every_tile(dev, dt, m, n, tile, slabs):
    slab, vec = (64, 8) if dt == "bf16" else (128, 16)
    k = slabs * slab - vec
    print(f"[case] fused ring {dt} {m}x{n}x{k} {tile}", flush=True)
    P = abft.Protected(DT[dt], m, n, k, 1, 1, device=dev, tau_mode=abft.ABFT_TAU_STAT, lam=10.0)
    desc = abft.describe_gemm(P.p, abft.ABFT_FUSED)
    assert desc.startswith(f"k_gemm_lowp {dt} {tile} on {m}x{n} k={k}"), desc
    A, As = operands(dev, dt, m, k, SEED % 9973, 0)
    B, Bs = operands(dev, dt, n, k, SEED % 9973 + 1, 0)
    P.A.copy_(As)
    P.Bt.copy_(Bs)
    P.encode()
    want = (A @ B.t()).float()
    P.gemm(abft.ABFT_FUSED)
    assert torch.equal(P.C[:m, :n], want)
    rep = P.verify_fused()
    assert (rep.status, rep.n_flag_c, rep.n_flag_r) == (abft.ABFT_OK, 0, 0)
    last = int((want[m - 1] >= 1).nonzero()[-1])                 # in the last tile row, near the last column
    first = int((want[0] >= 1).nonzero()[0])
    for i, j in ((m - 1, last), (0, first)):
        P.gemm_fault(i, j, 27, flags=abft.ABFT_FUSED)
        rep = P.verify_fused()
        assert rep.status == abft.ABFT_OK
        loc = abft.classify(P.p, rep)
        assert (loc.cls, loc.i, loc.j) == (abft.ABFT_CLS_DATA, i, j)
        abft.correct(P.p, P.C, loc)
        assert torch.equal(P.C[:m, :n], want)
