"""GPU parity of every instance of the product kernels where its pipeline differs: in the
steady loop (more stages than ring buffers by three or more, the last one ragged) and with
fewer stages than buffers.  The shapes name the kernel that the dispatch picks for them; the
CPU test of the rules asserts it.  Same oracles and tolerances as the other product tests."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_15682_amd import reqat
from paper_2606_15682_amd import workloads as wl
from tests.test_gpu_parity import DEV, GEMM_TOL, MX, NV, _rand, _w4a16_weights, log, run_gemm_case, run_w4a16

pytestmark = pytest.mark.gpu

# kernel, formats, M, N, K                 stages of 256 or 512 elements, ring buffers
W4A4 = [
    ("64x64", (NV, MX), 65, 1, 3200),              # 7 stages, ring of 4
    ("64x64", (NV,), 65, 1, 512),                  # a single stage
    ("64x64", (MX,), 65, 1, 640),
    ("64x128", (NV,), 1030, 2049, 1152),           # 5 stages, ring of 2
    ("64x128", (MX,), 513, 7001, 1152),
    ("64x128", (NV,), 65, 1, 128),                 # half a stage
    ("128x128", (NV,), 1543, 4113, 1152),          # 5 stages, ring of 2
    ("128x128", (MX,), 1543, 3001, 1408),
    ("128x128", (NV,), 385, 14001, 128),
    ("64x128 deep", (NV, MX), 1030, 1000, 1664),   # 7 stages, ring of 4
    ("64x128 deep", (MX,), 65, 1, 128),
    ("128x128 deep", (MX,), 1030, 2049, 1408),     # 6 stages, ring of 3
    ("128x128 deep", (MX,), 641, 3001, 256),
    # row-major and packed weights
    ("32x32", (NV, MX), 31, 4113, 3200),           # 7 stages, ring of 4
    ("32x32", (NV,), 31, 14001, 1152),
    ("32x32", (MX,), 31, 14001, 1536),
    ("32x128", (NV,), 31, 16401, 1408),            # 6 stages, ring of 3
    ("32x128", (MX,), 31, 14001, 1408),
    ("32x128", (NV, MX), 17, 16401, 128),
    ("64x32", (NV,), 50, 4113, 2688),              # 6 stages, ring of 3
    ("64x32", (MX,), 63, 1, 3456),
    ("64x32", (MX,), 61, 3601, 3456),
    ("64x32", (NV,), 50, 4113, 384),
    ("64x32", (MX,), 33, 4113, 768),
    ("64x64 few", (NV,), 50, 8225, 1664),          # 7 stages, ring of 4
    ("64x64 few", (MX,), 33, 8225, 1664),
    ("64x64 few", (NV, MX), 50, 4113, 128),
]

# gemm_w4a16_kernel: "split" adds partial sums of K in a second launch
W4A16 = [
    ("split", 4, 70, 16256), ("split", 13, 100, 12160), ("split", 16, 33, 16256), ("unsplit", 9, 16401, 384),
    ("split", 31, 100, 1152), ("unsplit", 20, 16500, 256), ("split", 33, 70, 1664), ("split", 50, 130, 6016),
]
W4A16_STRIDED = [("split", 13, 70, 12160), ("split", 40, 70, 1664), ("split", 31, 100, 1152)]
W4A16_SPECIAL = [("split", 9, 40, 16256), ("split", 27, 40, 1664), ("split", 40, 40, 1664)]


@pytest.mark.parametrize("fmt,M,N,K", [(f, *shape) for _, fmts, *shape in W4A4 for f in fmts])
def test_w4a4(fmt, M, N, K):
    log("w4a4 instances fmt=%d M=%d N=%d K=%d" % (fmt, M, N, K))
    run_gemm_case(fmt, M, N, K, seed=M + N + K, dist="student_t", all_points=M * N <= 60000)


@pytest.mark.parametrize("M,N,K", [shape for _, *shape in W4A16])
def test_w4a16(M, N, K):
    log("w4a16 instances M=%d N=%d K=%d" % (M, N, K))
    run_w4a16(_rand(M, K, M + N, "student_t", outliers=max(1, K // 100)), *_w4a16_weights(N, K, M + N))


@pytest.mark.parametrize("M,N,K", [shape for _, *shape in W4A16_STRIDED])
def test_w4a16_strided(M, N, K):
    """x read at ldx > K, y written at ldy > N, row-major and packed weights."""
    log("w4a16 strided M=%d N=%d K=%d" % (M, N, K))
    xb, (wc, ws) = _rand(M, K, 71 + M, "student_t", outliers=3), _w4a16_weights(N, K, 72 + N)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    wide = np.full((M, K + 8), 0x7F80, np.uint16)          # infinities beyond the rows
    wide[:, :K] = xb
    x = wl.from_bits(wide).to(DEV)[:, :K]
    y, yp = (torch.full((M, N + 3), float("nan"), dtype=torch.float32, device=DEV) for _ in range(2))
    reqat.gemm_w4a16(x, t(wc), t(ws), out=y[:, :N])
    reqat.gemm_w4a16_packed(x, reqat.pack_w4a16(t(wc), t(ws)), N, out=yp[:, :N])
    torch.cuda.synchronize()
    got = y.cpu().numpy().astype(np.float64)
    assert np.array_equal(got, yp.cpu().numpy(), equal_nan=True) and np.all(np.isnan(got[:, N:]))
    ref, aref = oracle.gemm_w4a16_points(xb, wc, ws, np.arange(M).repeat(N), np.tile(np.arange(N), M))
    assert np.all(np.abs(got[:, :N].reshape(-1) - ref) <= GEMM_TOL * aref)


@pytest.mark.parametrize("M,N,K", [shape for _, *shape in W4A16_SPECIAL])
def test_w4a16_special_values(M, N, K):
    """An infinity stays in its row, NaN blocks in their columns."""
    log("w4a16 special values M=%d N=%d K=%d" % (M, N, K))
    x = _rand(M, K, 91, "student_t", outliers=5)
    x[M - 1, 7] = 0x7F80
    wc, ws = _w4a16_weights(N, K, 91)
    wc[:, 3] |= 0x11                                      # no zero weight against the infinity
    ws[1, 0] = ws[N - 1, K // 32 - 1] = 0xFF
    ws[0, :] = 0
    run_w4a16(x, wc, ws)
