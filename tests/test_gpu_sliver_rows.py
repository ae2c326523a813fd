"""The carried column block of tall binary64 products (16384 operand rows and
more: a wave takes two operand rows and four chunks of k in a step) against
binary64 products of the stored checksum columns: an odd number of rows, one and
two checksum columns, and k of one vector, just under, at and just over a chunk
and a step of 512, so every clamped and skipped chunk occurs.  Both sides sum k
products in binary64 in some order: |C - ref| <= 2 (k + 1) u (|A||B|)."""
import pytest

torch = pytest.importorskip("torch")

from paper_0806_3121_amd import abft  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,bc", [(16385, 1), (16387, 2)])
@pytest.mark.parametrize("k", [2, 126, 130, 510, 514, 1150])
def test_carried_columns_of_tall_products(m, bc, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[case] tall carried columns m={m} bc={bc} k={k}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(7 * k + bc)
    n = 8
    P = abft.Protected(abft.ABFT_F64, m, n, k, 1, bc)
    assert "k_sliver1 carried columns" in abft.describe_gemm(P.p)
    P.A[:m].uniform_(-1, 1, generator=gen)
    P.Bt[:n].uniform_(-1, 1, generator=gen)
    P.encode()
    P.gemm()
    A, B = P.A[:m].cpu(), P.Bt[n:n + bc].cpu()
    bound = 2 * (k + 1) * 2.0 ** -53 * (A.abs() @ B.abs().t())
    assert ((P.C[:m, n:].cpu() - A @ B.t()).abs() <= bound).all()
    r = P.verify()
    assert r.n_flag_c == 0 and r.n_flag_r == 0
