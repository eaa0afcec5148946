"""GPU parity of the W4A4 product's plain tiles where several rounds of them, or
short rows, keep the dispatch from the deep ones: same oracle and tolerance as the
other product tests."""
import pytest

from tests.test_gpu_parity import MX, NV, log, run_gemm_case

pytestmark = pytest.mark.gpu


CASES = [
    ("64x128", (MX,), 130, 16400, 640),
    ("128x128", (MX,), 130, 22000, 1920),
    ("128x128", (NV,), 257, 19900, 384),
    ("64x128 deep", (NV,), 65, 8350, 1152),     # five stages, ring of four
    ("128x128 deep", (MX,), 65, 16400, 384),    # fewer stages than buffers
]


@pytest.mark.parametrize("fmt,M,N,K", [(f, M, N, K) for _, fmts, M, N, K in CASES for f in fmts])
def test_multiround_tiles(fmt, M, N, K):
    log("gemm tiles fmt=%d M=%d N=%d K=%d" % (fmt, M, N, K))
    run_gemm_case(fmt, M, N, K, seed=M + N + K, dist="student_t", all_points=False)
