"""NVFP4 quantize under a given g that is not a power of two, against the oracle bit for
bit: values at, and one bfloat16 step around, every scale bound 6 s g and rounding
midpoint of a block, zeros, subnormals and infinities among ordinary blocks, g with
many and with few significant bits and at the ends of the fast path's range."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_15682_amd import reqat
from paper_2606_15682_amd import workloads as wl
from tests.test_gpu_parity import DEV, NV, _rand, log

pytestmark = pytest.mark.gpu


def _bf16(v):
    """Nearest bfloat16 patterns (magnitudes; no infinities)."""
    u = np.asarray(v, np.float32).view(np.uint32)
    return np.minimum((u + 0x7FFF + ((u >> 16) & 1)) >> 16, 0x7F7F).astype(np.uint16)


def _edges(g, rows=96, cols=256):
    """Blocks whose largest value is a scale bound or next to one, the others midpoints or next to one."""
    rng = np.random.default_rng(int(g * 997) % 1000)
    s = np.array([(1 + m / 8) * 2.0 ** e for e in range(-7, 9) for m in range(8)])
    blocks = rows * cols // 16
    pick = rng.choice(s[s <= 448], blocks)[:, None]
    mid = np.array([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0, 0.0, 0.5, 6.0])
    v = rng.choice(mid, (blocks, 16)) * pick * g
    v[:, 0] = (6.0 * pick * g)[:, 0]
    b = _bf16(v).astype(np.int32) + rng.integers(-1, 2, v.shape)
    b = np.clip(b, 0, 0x7F7F).astype(np.uint16) | (rng.integers(0, 2, v.shape) << 15).astype(np.uint16)
    b[5] = 0                                              # a zero block
    b[6, 3] = 0x7F80                                      # an infinity
    b[7, 1:] = np.arange(15)                              # subnormals
    return b.reshape(rows, cols)


@pytest.mark.parametrize("g", [0.0123, 1.0 / 3.0, 3.5, 0.1875, 2.0 ** -100 * 1.1, 2.0 ** -101 * 1.1, 2.0 ** 99 * 1.7,
                               2.0 ** 101 * 1.3, 1.0000001])
@pytest.mark.parametrize("short", [1.0, 5.1, 1e5])        # g as calibrated, or too small for the largest blocks
def test_given_g(g, short):
    log("NVFP4 given g=%r / %r" % (g, short))
    x = _edges(float(np.float32(g)))
    g = float(np.float32(g / short))
    x = np.concatenate([x, _rand(70, 256, 3, "student_t", outliers=3)])
    codes, scales, _ = oracle.quantize(NV, x, g)
    c, s, _ = reqat.quantize(wl.from_bits(x).to(DEV), NV,
                             tensor_scale=torch.tensor([g], dtype=torch.float32, device=DEV))
    torch.cuda.synchronize()
    assert np.array_equal(s.cpu().numpy(), scales)
    assert np.array_equal(c.cpu().numpy(), codes)
