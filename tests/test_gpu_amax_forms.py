"""GPU test of the FP8 scale's pass: rows of every width it reads side by side
(one to sixty-four vectors across, ragged), in pieces, and rows that do not fill
the last load.  The one largest magnitude of an operand sits in turn at its
corners and in the middle; it alone decides the scale exponent, and with it
every code, which must be the oracle's.  Infinities and NaN beside it take no
part in the scale."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_0806_3121_amd import abft, synth  # noqa: E402

pytestmark = pytest.mark.gpu

SEED = synth.BASE_SEED + 233


@pytest.mark.parametrize("rows,k", [(1, 16), (3, 16), (130, 32), (67, 48), (33, 80), (65, 112), (31, 128), (17, 144),
                                    (257, 256), (9, 272), (40, 1040), (11, 2048), (7, 2064), (3, 16400)])
def test_the_largest_magnitude_is_found_wherever_it_is(orc, rows, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P = abft.Protected(abft.ABFT_FP8_E4M3, rows, rows, k, 1, 1)
    X0 = synth.uniform(SEED, synth.STREAM_A, rows, k, np.float32)
    for i, l in {(0, 0), (rows - 1, k - 1), (rows - 1, 0), (0, k - 1), (rows // 2, k // 2)}:
        print(f"[case] amax {rows}x{k} at ({i},{l})", flush=True)
        X = X0.copy()
        X[i, l] = -37.5
        X[i, l - 1 if l else 1] = np.inf
        codes = orc.to_e4m3_codes(np.ldexp(X.astype(np.float64), 3).astype(np.float32))    # 37.5 * 2^3 <= 448 < 37.5 * 2^4
        for which, dst in ((0, P.A), (1, P.Bt)):
            abft.quantize(P.p, which, torch.from_numpy(X).cuda(), dst, P.ws)
            assert np.array_equal(dst.cpu().numpy(), codes)
        abft.quantize_encode(P.p, torch.from_numpy(X0).cuda(), torch.from_numpy(X).cuda(), P.A, P.Bt, P.ws)
        assert np.array_equal(P.Bt.cpu().numpy(), codes)
