"""GPU test of the verification's passes over C_f: column sums by partitions and
by whole residues, row sums by a wave per row (every checksum width that divides
its vectors), by a block per row (rows not on 16-byte boundaries) and strided,
both directions in one read, and the b = 1 tile sums, at ragged sizes.

C_f holds integers that satisfy every relation, the thresholds are exact (0),
and a few entries in distinct relations are changed: the failed relations and
their residuals must be exactly those of the changed entries."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_0806_3121_amd import abft, synth  # noqa: E402

pytestmark = pytest.mark.gpu

SEED = synth.BASE_SEED + 191

CASES = [
    # dtype, m, n, br, bc, ldc - (n + bc)
    ("f64", 700, 515, 1, 1, 0),      # tile sums, ragged tiles
    ("f32", 257, 1030, 1, 1, 1),     # ldc a multiple of 4: 16-byte rows
    ("f32", 300, 260, 1, 1, 0),      # 261 columns: rows off 16 bytes, column partitions and a block per row
    ("f64", 640, 1026, 2, 2, 0),     # a wave per row, two residues in a vector
    ("f32", 390, 1028, 3, 2, 2),     # residues folded inside a vector
    ("f32", 390, 1028, 3, 4, 0),
    ("f64", 512, 1032, 8, 8, 0),
    ("f32", 1600, 1056, 32, 32, 0),  # 50 groups: partitions with a remainder
    ("f64", 544, 1056, 16, 32, 1),   # odd ldc: a block per row
    ("f64", 480, 420, 48, 20, 0),    # strided rows (20 divides no power of two)
    ("f64", 320, 320, 64, 64, 0),    # few groups: whole residues
    ("f64", 1536, 1536, 256, 256, 0),  # both directions in one read
    ("f32", 24, 2048, 3, 512, 0),    # strided rows, wide blocks
    ("f64", 1, 2, 1, 1, 1),          # the smallest
]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    abft.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_exactly_the_changed_relations_fail(dev, case):
    dt, m, n, br, bc, pad = case
    print(f"[case] verify split {case}", flush=True)
    f32 = dt == "f32"
    D = synth.uniform_ints(SEED, synth.STREAM_A, m, n, -3, 3)
    C = np.zeros((m + br, n + bc))
    C[:m, :n] = D
    C[m:, :n] = D.reshape(m // br, br, n).sum(axis=0)
    C[:, n:] = C[:, :n].reshape(m + br, n // bc, bc).sum(axis=1)
    # changed entries in distinct column relations and distinct row relations
    want_c, want_r = {}, {}
    for t in range(40):
        i = synth.randint(SEED, synth.STREAM_FLIP, 2 * t, m + br)
        j = synth.randint(SEED, synth.STREAM_FLIP, 2 * t + 1, n + bc)
        r, c = (i if i < m else i - m) % br, (j if j < n else j - n) % bc
        if (r, j) in want_c or (i, c) in want_r:
            continue
        C[i, j] += t + 1
        want_c[(r, j)] = (t + 1.0) * (1 if i < m else -1)
        want_r[(i, c)] = (t + 1.0) * (1 if j < n else -1)
    p = abft.problem(abft.ABFT_F32 if f32 else abft.ABFT_F64, m, n, 16, br, bc, ldc=n + bc + pad,
                     tau_mode=abft.ABFT_TAU_EXACT)
    buf = torch.full((m + br, n + bc + pad), float("nan"), dtype=torch.float32 if f32 else torch.float64, device=dev)
    buf[:, :n + bc] = torch.from_numpy(C).to(dev)
    ws = torch.zeros(abft.workspace_size(p), dtype=torch.uint8, device=dev)
    host = abft.new_report_buffer()
    for verify in (abft.verify, abft.verify_noalloc):
        host.fill_(255)
        verify(p, buf, ws, host_out=host)
        torch.cuda.synchronize()
        rep = abft.read_report(host)
        assert (rep.n_flag_c, rep.n_flag_r, rep.n_nonfinite, rep.status) == (len(want_c), len(want_r), 0, 0)
        assert {(a, b): d for a, b, d, _ in rep.flags_c()} == want_c
        assert {(a, b): d for a, b, d, _ in rep.flags_r()} == want_r
