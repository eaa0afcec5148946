"""CPU model of the KV4 kernel's rounding without a shift (no GPU, no oracle).

An unshifted d is a bfloat16 value; with a power-of-two global scale H = s g / 2
has at most four significant bits.  The kernel takes c = rint(q), q = RN(d r + 3072)
- 3072 in FP32 (r the reciprocal of H, within one ulp), and trusts every c.  Here
that arithmetic runs for every bfloat16 magnitude up to 7 H, every E4M3
significand (subnormal scales too) and exponents up to the ends of the range,
against exact integer rounding."""
from fractions import Fraction

import numpy as np
import pytest


def _exact(d, h):
    """Nearest integers to |d| / h, ties to even."""
    out = np.empty(d.size, np.int64)
    for i, v in enumerate(d):
        q = Fraction(float(abs(v))) / h
        n = int(q)
        rem = 2 * (q - n)
        out[i] = n + (rem > 1 or (rem == 1 and n % 2 == 1))
    return out


@pytest.mark.parametrize("e", [-126, -125, -60, -7, 0, 40, 119])
def test_codes_of_every_bfloat16(e):
    for h in range(8, 16):                                # h / 8: every E4M3 significand, 1.000 to 1.111
        H = np.float32(h / 8.0 * 2.0 ** e)
        top = min(int((np.float32(7.0) * H).view(np.uint32)) >> 16, 0x7F7F)
        low = max(top - 128 * 12, 0)                      # twelve binades down: q < 2^-8 below that
        d = (np.arange(low, top + 1, dtype=np.uint32) << 16).view(np.float32)
        d = d[d <= np.float32(7.0) * H]
        d = np.concatenate([d, -d, np.array([0.0, -0.0, 2.0 ** -133, -2.0 ** -133], np.float32)])
        want = _exact(d, Fraction(float(H)))
        r0 = np.float32(1.0) / H
        for r in (r0, np.nextafter(r0, np.float32(0)), np.nextafter(r0, np.float32(np.inf))):
            # the FMA: the product is exact in FP64 (8 + 24 bits), the sum there to 2^-41
            q = (d.astype(np.float64) * np.float64(r) + 3072.0).astype(np.float32) - np.float32(3072.0)
            c = np.copysign(np.rint(q), d)
            assert np.array_equal(np.abs(c).astype(np.int64), want), (h, e)
            assert np.array_equal(np.signbit(c), np.signbit(d))
            assert np.abs(c).max() <= 7
