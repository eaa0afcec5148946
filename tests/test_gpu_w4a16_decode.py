"""GPU parity of the W4A16 decode kernel that keeps K inside a workgroup (M <= 16, few
weight rows): every row count around its groups of four, K of fewer chunks than waves, of
one and of several chunks per wave, ragged N, NaN blocks and infinities, at the sizes
its rule takes.  Same oracle and tolerance as the other W4A16 tests."""
import pytest

from tests.test_gpu_parity import _rand, _w4a16_weights, log, run_w4a16

pytestmark = pytest.mark.gpu


ROWS, SHAPES = [1, 3, 4, 5, 8, 9, 13, 16], [(17, 128), (100, 896), (33, 1152), (48, 4736)]


@pytest.mark.parametrize("M", ROWS)
@pytest.mark.parametrize("N,K", SHAPES)
def test_decode_rows(M, N, K):
    log("w4a16 decode M=%d N=%d K=%d" % (M, N, K))
    run_w4a16(_rand(M, K, M + N, "student_t", outliers=max(1, K // 100)), *_w4a16_weights(N, K, M + N))


@pytest.mark.parametrize("M", [2, 7, 14])
def test_special_values(M):
    """An infinity stays in its row, NaN blocks in their columns."""
    x = _rand(M, 512, 91, "student_t", outliers=5)
    x[M - 1, 7] = 0x7F80
    wc, ws = _w4a16_weights(40, 512, 91)
    wc[:, 3] |= 0x11                                      # no zero weight against the infinity
    ws[1, 0] = ws[39, 15] = 0xFF
    ws[0, :] = 0
    run_w4a16(x, wc, ws)
