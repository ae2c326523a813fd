"""GPU test of the weighted encode in one read (enough relations that each
lane sums whole residues, or a single block): checksum rows against the
oracle's weighted sums, and the thresholds built from the row norms of the
same read.  Ragged strips (k / V not a multiple of 64), residues and blocks
that leave partial groups of four, and the streamed operand beyond the caches.
A C_f of NaN fails every group, so the report lists 64 thresholds of each
direction.

Tolerances: a checksum entry sums G products in binary64 (G 2^-52 times the
sum of magnitudes, below 2 G here), rounded once to binary32 for binary32; a
threshold carries a few (k + G) 2^-53."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import weighted as wo  # noqa: E402
from paper_0806_3121_amd import abft, synth  # noqa: E402

pytestmark = pytest.mark.gpu

SEED = synth.BASE_SEED + 171
U32 = 2.0 ** -24

CASES = [
    # dtype, m, n, k, br, bc, fr, fc
    ("f64", 910, 6, 8066, 130, 6, 2, 1),      # 7 blocks; 4033 vectors: 64 strips, one lane in the last; B one block
    ("f64", 264, 130, 8066, 132, 130, 3, 4),  # two blocks, one block
    ("f64", 3, 1, 2, 3, 1, 1, 2),             # one block each, one vector
    ("f32", 650, 10, 16132, 130, 10, 4, 2),
    ("f64", 4096, 2, 8194, 64, 1, 1, 1),      # 268 MB: streamed loads
]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    abft.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_checksums_and_thresholds_match_oracle(dev, case):
    dt, m, n, k, br, bc, fr, fc = case
    print(f"[case] weighted encode {case}", flush=True)
    f32 = dt == "f32"
    npdt = np.float32 if f32 else np.float64
    A = synth.uniform(SEED, synth.STREAM_A, m, k, npdt)
    Bt = synth.uniform(SEED, synth.STREAM_B, n, k, npdt)
    Wr = 0.5 + (synth.uniform(SEED, synth.STREAM_X, fr, m // br) + 1) / 2
    Wc = 0.5 + (synth.uniform(SEED, synth.STREAM_PICK, fc, n // bc) + 1) / 2
    P = abft.WProtected(m, n, k, br, bc, Wr, Wc, device=dev, dtype=abft.ABFT_F32 if f32 else abft.ABFT_F64)
    P.A[:m], P.Bt[:n] = torch.from_numpy(A).to(dev), torch.from_numpy(Bt).to(dev)
    P.encode()
    Af, Bf = wo.wencode(A.astype(np.float64), np.ascontiguousarray(Bt.T).astype(np.float64), Wr, Wc, br, bc)
    for got, want, G in ((P.A[m:].cpu().numpy(), Af[m:], m // br), (P.Bt[n:].cpu().numpy(), Bf[:, n:].T, n // bc)):
        assert np.abs(got - want).max() <= 2 * G * (G * 2.0 ** -52 + f32 * U32)
    # the operands as stored (binary32 checksum rows rounded once), as the kernels' norms see them
    Af, Bf = P.A.cpu().numpy().astype(np.float64), np.ascontiguousarray(P.Bt.cpu().numpy().T).astype(np.float64)
    kw = dict(u_acc=U32, u_st=U32) if f32 else {}
    tc, tr = wo.wtau_det(Af, Bf, m, n, br, bc, Wr, Wc, **kw)
    P.C.fill_(float("nan"))
    rep = P.verify()
    assert rep.n_fail_c == br * P.N and rep.n_fail_r == P.M * bc
    for i, j, _, tau in rep.groups_c(fr):
        assert all(abs(tau[r] - tc[r, i, j]) <= 1e-10 * tc[r, i, j] for r in range(fr)), (i, j, tau, tc[:, i, j])
    for x, jj, _, tau in rep.groups_r(fc):
        assert all(abs(tau[c] - tr[x, c, jj]) <= 1e-10 * tr[x, c, jj] for c in range(fc)), (x, jj, tau, tr[x, :, jj])
