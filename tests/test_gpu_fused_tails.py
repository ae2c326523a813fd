"""GPU test of the fused epilogue behind a masked last slab: every direct
binary64 / binary32 tile that a fused product of a ragged k can run on, and the
same tiles with whole slabs, through the checks of test_gpu_fused (C bit for bit
that of the unfused product and the oracle's, a clean fused verification, an
accumulator flipped in the last row and column and elsewhere, found and
corrected from the product's own partial sums)."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_fused import dev  # noqa: E402,F401
from test_gpu_fused import test_fused_clean_and_accumulator_flips as _check  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [
    ("f64", 601, 503, 250, "k_gemm_mfma2 f64 96x96"),
    ("f64", 2001, 1503, 1234, "k_gemm_mfma2 f64 128x96"),
    ("f64", 601, 503, 256, "k_gemm_mfma2 f64 96x96"),
    ("f32", 513, 512, 1000, "k_gemm_mfma2 f32 128x128"),
    ("f32", 4000, 1990, 156, "k_gemm_mfma2 f32 256x128"),
    ("f32", 513, 512, 1024, "k_gemm_mfma2 f32 128x128"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c[:4])))
def test_fused_clean_and_accumulator_flips(dev, orc, case):  # noqa: F811
    _check(dev, orc, case)
