"""GPU parity of the W4A16 product's tile kernels (M > 32), row-major and packed weights,
at the shapes where each can go wrong: rows and columns one past a tile or a 16-row
group, one stage, fewer stages than ring buffers, odd and even numbers of stages, x with
a row stride, y in rows that are not 16-byte aligned, NaN scale bytes and infinities.
Against the FP64 product of the oracle with the tolerance of the other W4A16 tests
(run_w4a16 compares packed and row-major bit for bit), and, for the tiles that small
oracles do not reach, against the 64-bit product of torch."""
import numpy as np
import pytest
import torch

from paper_2606_15682_amd import reqat
from tests.test_gpu_parity import DEV, GEMM_TOL, _rand, _w4a16_weights, log, run_w4a16

pytestmark = pytest.mark.gpu


# 64 x 64 tiles (stages of 128); the dispatch's picks are asserted by the CPU test of its rules
SMALL = [(65, 33, 128), (129, 130, 256), (200, 65, 384), (130, 100, 640), (65, 1, 1152)]


@pytest.mark.parametrize("M,N,K", SMALL)
def test_small_tiles(M, N, K):
    log("w4a16 tiles M=%d N=%d K=%d" % (M, N, K))
    run_w4a16(_rand(M, K, M + N, "student_t", outliers=max(1, K // 100)), *_w4a16_weights(N, K, M + N))


def test_special_values():
    """NaN blocks and an infinity of x reach their own columns and rows alone."""
    x = _rand(70, 512, 91, "student_t", outliers=5)
    x[3, 7] = 0x7F80
    wc, ws = _w4a16_weights(40, 512, 91)
    wc[:, 3] |= 0x11                                      # no zero weight against the infinity
    ws[1, 0] = ws[39, 15] = 0xFF
    ws[0, :] = 0
    run_w4a16(x, wc, ws)


def _dequantized(wc, ws):
    grid = torch.tensor([0, 0.5, 1, 1.5, 2, 3, 4, 6], dtype=torch.float64, device=DEV)
    c = torch.stack([wc & 15, wc >> 4], -1).reshape(wc.shape[0], -1).long()
    v = torch.where(c >= 8, -1.0, 1.0).double() * grid[c & 7]
    e = ((ws.long() - 127 + 1023) << 52).view(torch.float64)
    return (v.reshape(len(ws), -1, 32) * e[:, :, None]).reshape(len(ws), -1)


LARGE = [("64x128", 65, 12000, 384, "f32"), ("64x128", 100, 17003, 1152, "bf16"), ("64x128", 300, 27700, 256, "f32"),
         ("64x128", 385, 5105, 1152, "bf16"), ("64x128", 65, 8225, 128, "f32"),
         ("128x128", 700, 10001, 1280, "bf16"), ("128x128", 641, 9001, 768, "f32"),
         ("128x128x8", 200, 16001, 640, "f32"), ("128x128x8", 770, 4113, 896, "bf16"), ("128x128x8", 770, 4113, 1024, "f32")]


@pytest.mark.parametrize("M,N,K,out", [case for _, *case in LARGE])
def test_large_tiles(M, N, K, out):
    log("w4a16 large tiles M=%d N=%d K=%d" % (M, N, K))
    g = torch.Generator(device=DEV).manual_seed(M + N)
    wide = torch.randn((M, K + 8), generator=g, device=DEV, dtype=torch.bfloat16)
    x = wide[:, :K]                                       # rows 16 bytes apart beyond K
    wc = torch.randint(0, 256, (N, K // 2), generator=g, device=DEV, dtype=torch.uint8)
    ws = torch.randint(110, 140, (N, K // 32), generator=g, device=DEV, dtype=torch.uint8)
    dt = torch.float32 if out == "f32" else torch.bfloat16
    big = torch.full((M, N + 3), 7.0, dtype=dt, device=DEV)
    y = reqat.gemm_w4a16(x, wc, ws, out_dtype=dt, out=big[:, :N])
    dense = reqat.gemm_w4a16_packed(x, reqat.pack_w4a16(wc, ws), N, out_dtype=dt)
    torch.cuda.synchronize()
    assert torch.equal(y, dense) and bool((big[:, N:] == 7.0).all())
    for n in range(0, N, 4096):
        w = _dequantized(wc[n:n + 4096], ws[n:n + 4096])
        ref = torch.mm(x.double(), w.t())
        mag = torch.mm(x.double().abs(), w.t().abs())
        tol = GEMM_TOL * mag + (0 if out == "f32" else 2.0 ** -8) * ref.abs()
        assert bool(((dense[:, n:n + 4096].double() - ref).abs() <= tol).all())
        # FP32 sums of K exact products (each MFMA adds eight): half an ulp an addition
        if out == "f32":
            assert bool(((dense[:, n:n + 4096].double() - ref).abs() <= K * 2.0 ** -24 * mag).all())
