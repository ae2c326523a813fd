"""GPU parity of the binary64 / binary32 tiles picked by rounds (four slabs of
k and more) against the CPU oracle: the small tiles, and every direct tile
with a k that is not a multiple of the 128-byte slab, at remainders of one
vector and one short of a slab, with ragged m and n so every tile has partial
edge tiles.  Each case names the tile that must run.  The accumulating panel
product of the same shapes adds to a C_f of known values.

Tolerances as for the other tiles: max|C - C_oracle| / max|C_oracle| <= 1e-12
(binary64) or 1e-5 (binary32)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_0806_3121_amd import abft, synth  # noqa: E402

pytestmark = pytest.mark.gpu

SEED = synth.BASE_SEED + 151
DT = {"f64": abft.ABFT_F64, "f32": abft.ABFT_F32}

CASES = [
    ("f64", 300, 260, 64, "32x32"),
    ("f64", 400, 390, 78, "32x32"),       # remainder one vector short of a slab
    ("f64", 1000, 990, 64, "64x64"),
    ("f64", 900, 1000, 66, "64x64"),      # remainder of one vector
    ("f64", 1500, 1490, 98, "96x96"),
    ("f64", 2001, 1503, 82, "128x96"),
    ("f32", 300, 260, 128, "32x32"),
    ("f32", 400, 390, 156, "32x32"),
    ("f32", 1000, 990, 128, "64x64"),
    ("f32", 900, 1000, 132, "64x64"),
    ("f32", 2000, 1990, 132, "128x128"),
    ("f32", 4000, 1990, 156, "256x128"),
]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    abft.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_tile_matches_oracle(dev, orc, case):
    dt, m, n, k, tile = case
    print(f"[case] rounds tile {case}", flush=True)
    npdt = np.float64 if dt == "f64" else np.float32
    A = synth.uniform(SEED, synth.STREAM_A, m, k, npdt)
    Bt = synth.uniform(SEED, synth.STREAM_B, n, k, npdt)
    mode = abft.ABFT_TAU_DET if dt == "f64" else abft.ABFT_TAU_STAT
    P = abft.Protected(DT[dt], m, n, k, 1, 1, device=dev, tau_mode=mode, lam=10.0)
    desc = abft.describe_gemm(P.p)
    assert desc.startswith(f"k_gemm_mfma2 {dt} {tile} on {m}x{n} k={k}"), desc
    P.A[:m], P.Bt[:n] = torch.from_numpy(A).to(dev), torch.from_numpy(Bt).to(dev)
    P.encode()
    P.gemm()
    Af, Bf = orc.encode(A.astype(np.float64), np.ascontiguousarray(Bt.T).astype(np.float64), 1, 1,
                        store_f32=dt == "f32")
    ref = orc.gemm(Af, Bf)
    tol = 1e-12 if dt == "f64" else 1e-5
    assert np.abs(P.C.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()
    rep = P.verify()
    assert rep.n_flag_c == 0 and rep.n_flag_r == 0
    # the whole k as one accumulating panel
    P.C.fill_(2.0)
    abft.gemm_panel(P.p, P.A, P.Bt, P.C, 0, k, abft.ABFT_ACCUMULATE)
    assert np.abs(P.C.cpu().numpy() - (ref + 2.0)).max() <= tol * np.abs(ref + 2.0).max()


@pytest.mark.parametrize("dt,m,n,k", [("f64", 900, 1000, 66), ("f32", 400, 390, 156)])
def test_infinities_stay_in_their_rows(dev, dt, m, n, k):
    """An infinite operand entry near the end of k reaches its own row (or
    column) only: the masked part of the last slab multiplies nothing."""
    print(f"[case] infinity at the end of k {dt} {m}x{n}x{k}", flush=True)
    npdt = np.float64 if dt == "f64" else np.float32
    A = torch.from_numpy(np.abs(synth.uniform(SEED, synth.STREAM_A, m, k, npdt)) + 0.5).to(dev)
    Bt = torch.from_numpy(np.abs(synth.uniform(SEED, synth.STREAM_B, n, k, npdt)) + 0.5).to(dev)
    A[7, k - 1] = float("inf")
    Bt[n - 2, k - 2] = float("inf")
    p = abft.problem(DT[dt], m, n, k, 1, 1, ldc=n)
    C = torch.zeros(m, n, dtype=A.dtype, device=dev)
    abft.gemm(p, A, Bt, C, None, abft.ABFT_PLAIN)
    inf = torch.isinf(C)
    want = torch.zeros_like(inf)
    want[7, :] = True
    want[:, n - 2] = True
    assert torch.equal(inf, want) and not torch.isnan(C).any()
