"""NVFP4 codes, scales and computed g against the oracle around the size up to which every
workgroup reads the whole tensor for its amax: dense and strided rows, the amax in the
first and the last element, NaN and infinities that must not count, all zeros."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_15682_amd import reqat
from paper_2606_15682_amd import workloads as wl
from tests.test_gpu_parity import DEV, NV, _rand, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pad", [0, 16])
@pytest.mark.parametrize("rows,cols", [(1, 16), (3, 1552), (32, 2048), (33, 2048), (96, 2048), (97, 2048), (12, 16384)])
@pytest.mark.parametrize("kind", ["plain", "first", "last", "nonfinite", "zero"])
def test_amax(rows, cols, pad, kind):
    log("NVFP4 small amax %dx%d pad=%d %s" % (rows, cols, pad, kind))
    x = _rand(rows, cols, rows + cols, "student_t")
    if kind == "first":
        x[0, 0] = 0xC580                                  # -4096
    elif kind == "last":
        x[-1, -1] = 0x4580
    elif kind == "nonfinite":
        x[0, 1], x[-1, 0], x[rows // 2, 3] = 0x7FC0, 0xFF80, 0x7F80
    elif kind == "zero":
        x[:] = 0
    codes, scales, g = oracle.quantize(NV, x)
    wide = np.full((rows, cols + pad), 0x7F00, np.uint16)  # a larger value beyond the rows
    wide[:, :cols] = x
    c, s, gg = reqat.quantize(wl.from_bits(wide).to(DEV)[:, :cols], NV)
    torch.cuda.synchronize()
    assert float(gg.cpu()[0]) == g
    assert np.array_equal(s.cpu().numpy(), scales) and np.array_equal(c.cpu().numpy(), codes)
