"""CPU model of the NVFP4 quantizer's arithmetic under a g that is not a power of two,
against the oracle (its general rule): scale bytes and codes from FP32 quotients
snapped to a few bits and the sign of an FP32 residual, with the reciprocals one ulp
either way, on blocks at and next to every scale bound and midpoint."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_quant_given import _edges
from tests.test_gpu_parity import NV

F = np.float32


def _fma(a, b, c):
    # the product of two FP32 is exact in long double (64 bits); where c cancels, so is the sum
    return (np.longdouble(a) * np.longdouble(b) + np.longdouble(c)).astype(F)


def _snap(y, half, mask):
    return ((y.view(np.uint32) + np.uint32(half)) & np.uint32(mask)).view(F)


def _model(x, g, ulp):
    """(blocks the path takes, scale bytes, codes); ulp moves both reciprocals."""
    rcp = lambda v: np.nextafter(F(1) / v, F(np.inf) * ulp, dtype=F) if ulp else F(1) / v
    xf = (x.astype(np.uint32) << 16).view(F).reshape(-1, 16)
    a, g = np.abs(xf).max(1), F(g)
    g6 = F(6) * g
    c = _snap(a * rcp(g6), 0x80000, 0xFFF00000)
    up = _fma(-c, _fma(F(6), g, -g6), _fma(-c, g6, a)) > 0
    sb = (c.view(np.uint32) >> 20) + up
    ok = (a > 0) & np.isfinite(a) & (c >= F(2.0 ** -6)) & (c <= F(2.0 ** 20))
    sb = np.minimum(sb, 0x7E + 960)
    s = (sb.astype(np.uint32) << 20).view(F)
    h = s * g
    low = _fma(s, g, -h)[:, None]
    c = _snap(xf * rcp(h)[:, None], 0x100000, 0xFFE00000)
    e = _fma(-c, low, _fma(-c, h[:, None], xf))
    n = np.clip(e * F(2.0 ** 126), -F(2.0 ** -6), F(2.0 ** -6))
    y = np.copysign(_fma(np.abs(c), n, c), xf)
    code = np.zeros(y.shape, np.uint8)
    for i, mid in enumerate((0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0)):     # ties to the even code
        code += np.abs(y) >= mid if i & 1 else np.abs(y) > mid
    return ok, sb - 960, code | (np.signbit(y) << 3).astype(np.uint8)


@pytest.mark.parametrize("ulp", [0, 1, -1])
@pytest.mark.parametrize("short", [1.0, 5.1])             # g as calibrated, or too small for the largest blocks
@pytest.mark.parametrize("g", [0.0123, 1.0 / 3.0, 3.5, 0.1875, 2.0 ** -100 * 1.1, 2.0 ** 99 * 1.7, 1.0000001])
def test_every_block_the_path_takes(g, short, ulp):
    x = _edges(float(F(g)), rows=600)
    g = float(F(g / short))
    codes, scales, _ = oracle.quantize(NV, x, g)
    with np.errstate(all="ignore"):
        ok, sb, code = _model(x, g, ulp)
    ref = np.stack([codes & 15, codes >> 4], -1).reshape(-1, 16)
    assert ok.mean() > 0.85
    assert np.array_equal(sb[ok], scales.reshape(-1)[ok])
    assert np.array_equal(code[ok], ref[ok])
