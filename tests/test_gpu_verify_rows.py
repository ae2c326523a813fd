"""GPU test of the row relations' forms beside those of test_gpu_verify_split: a
row shared by the block's waves (few long rows, every width that divides a
vector, ragged ends), several residues per thread (blocks of one to nine per row,
widths that are multiples of a vector and no power of two), and many failing
relations, which are counted exactly whichever lane finds them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_0806_3121_amd import abft  # noqa: E402
from test_gpu_verify_split import dev  # noqa: E402,F401
from test_gpu_verify_split import test_exactly_the_changed_relations_fail as _check  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, m, n, br, bc, ldc - (n + bc)
    ("f64", 10, 4099, 2, 1, 0), ("f64", 6, 2050, 3, 2, 0), ("f64", 33, 8192, 1, 4, 0), ("f64", 32, 2080, 16, 32, 0),
    ("f32", 10, 4101, 2, 1, 2), ("f32", 2, 16386, 1, 2, 0), ("f32", 5, 4100, 1, 4, 0), ("f32", 8, 4128, 8, 32, 0),
    ("f64", 1023, 2048, 1, 2, 0), ("f64", 1030, 2048, 1, 2, 0),       # either side of the line between the two
    ("f64", 12, 66, 3, 66, 0), ("f64", 12, 132, 3, 66, 0), ("f32", 20, 300, 4, 100, 0), ("f32", 20, 400, 4, 100, 0),
    ("f32", 9, 340, 3, 68, 0), ("f64", 30, 630, 5, 70, 0), ("f32", 40, 192, 8, 12, 0), ("f32", 40, 198, 8, 18, 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_exactly_the_changed_relations_fail(dev, case):  # noqa: F811
    _check(dev, case)


@pytest.mark.parametrize("dt,m,n,br,bc", [("f64", 60, 96, 2, 8), ("f32", 60, 96, 3, 16), ("f32", 8, 8192, 4, 2),
                                          ("f32", 24, 204, 4, 68), ("f64", 50, 200, 1, 1)])
def test_every_relation_fails(dev, dt, m, n, br, bc):  # noqa: F811
    """Data of ones with carried blocks of zeros: every relation over data fails, none over carried entries alone."""
    print(f"[case] every relation fails {dt} {m}x{n} {br},{bc}", flush=True)
    vec = 2 if dt == "f64" else 4
    ldc = (n + bc + vec - 1) // vec * vec
    p = abft.problem(abft.ABFT_F64 if dt == "f64" else abft.ABFT_F32, m, n, 16, br, bc, ldc=ldc,
                     tau_mode=abft.ABFT_TAU_EXACT)
    C = torch.zeros(m + br, ldc, dtype=torch.float64 if dt == "f64" else torch.float32, device=dev)
    C[:m, :n] = 1.0
    ws = torch.zeros(abft.workspace_size(p), dtype=torch.uint8, device=dev)
    host = abft.new_report_buffer()
    abft.verify(p, C, ws, host_out=host)
    torch.cuda.synchronize()
    rep = abft.read_report(host)
    assert (rep.n_flag_c, rep.n_flag_r) == (br * n, m * bc)
    assert {d for _, _, d, _ in rep.flags_c()} == {float(m // br)}
    assert {d for _, _, d, _ in rep.flags_r()} == {float(n // bc)}
    rows = [(a, b) for a, b, _, _ in rep.flags_r()]
    assert len(set(rows)) == min(64, m * bc) and all(0 <= a < m and 0 <= b < bc for a, b in rows)
