"""GPU parity of the W4A4 product's tiles for 17 to 64 rows, row-major and packed
weights (run_gemm_case compares the two bit for bit), at the shapes where each can
go wrong: rows and columns one past a tile or a 16-row group, K that ends inside
a stage (384, 640, 2176 elements against stages of 256 and 512) or inside a
256-element unit of the image, fewer stages than ring buffers.  Same oracle and
tolerance as the other product tests."""
import pytest

from tests.test_gpu_parity import MX, NV, log, run_gemm_case

pytestmark = pytest.mark.gpu

# (tile, formats, M, N, K): the dispatch picks the named tile (asserted by the CPU test of its rules)
CASES = [
    ("skinny", (NV, MX), 17, 4113, 2176),
    ("32x32", (NV, MX), 32, 4200, 2944),        # six stages of 512, the last three quarters full
    ("32x128", (NV, MX), 31, 32000, 640),       # three stages of 256, ring of three
    ("64x32", (NV,), 64, 4113, 640),            # two stages
    ("64x64 few", (MX,), 64, 4113, 640),        # K shared by four sets of waves
    ("skinny", (NV,), 33, 4100, 2432),
    ("64x32", (MX,), 33, 4100, 2432),
    ("64x64 few", (NV, MX), 50, 8300, 640),
    ("64x64 few", (NV, MX), 64, 8225, 2176),
]


@pytest.mark.parametrize("fmt,M,N,K", [(f, M, N, K) for _, fmts, M, N, K in CASES for f in fmts])
def test_decode_tiles(fmt, M, N, K):
    log("decode tiles fmt=%d M=%d N=%d K=%d" % (fmt, M, N, K))
    run_gemm_case(fmt, M, N, K, seed=M + N + K, dist="student_t", all_points=False)


def test_one_short_stage():
    """K = 128: one stage, half full, half a unit of the image."""
    run_gemm_case(MX, 64, 4200, 128, seed=9, dist="student_t", all_points=False)
