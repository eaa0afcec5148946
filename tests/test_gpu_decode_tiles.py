"""GPU parity of the W4A4 product's tiles for 17 to 64 rows, row-major and packed
weights (run_gemm_case compares the two bit for bit), at the shapes where each can
go wrong: rows and columns one past a tile or a 16-row group, K that ends inside
a stage (384, 640, 2176 elements against stages of 256 and 512) or inside a
256-element unit of the image, fewer stages than ring buffers.  Same oracle and
tolerance as the other product tests."""
import pytest

from tests.test_gpu_parity import MX, NV, log, run_gemm_case

pytestmark = pytest.mark.gpu

# the dispatch's costs pick the named tile for both formats
CASES = [
    (17, 4113, 2176),       # 32 x 32: five stages of 512, the last a quarter full
    (32, 4200, 2944),
    (31, 32000, 640),       # 32 x 128: three stages of 256, ring of three
    (64, 4113, 640),        # 64 x 32: two stages
    (33, 4100, 2432),
    (50, 8300, 640),        # 64 x 64 with K shared by four sets of waves
    (64, 8225, 2176),
]


@pytest.mark.parametrize("fmt", [NV, MX])
@pytest.mark.parametrize("M,N,K", CASES)
def test_decode_tiles(fmt, M, N, K):
    log("decode tiles fmt=%d M=%d N=%d K=%d" % (fmt, M, N, K))
    run_gemm_case(fmt, M, N, K, seed=M + N + K, dist="student_t", all_points=False)


def test_one_short_stage():
    """64 x 32 tiles with K = 128: one stage, a quarter full, half a unit of the image."""
    run_gemm_case(MX, 64, 4200, 128, seed=9, dist="student_t", all_points=False)
