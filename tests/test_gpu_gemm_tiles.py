"""GPU parity of the W4A4 product's tile kernels for M > 64 rows, at the shapes
where each can go wrong: one row or column past a tile, K that ends inside a
stage (128, 384, 640, 1152, 2176 elements against stages of 256 and 512) or
inside a group of scale bytes, a single stage, more stages than ring buffers,
rows of y that are not 8-byte aligned.  Same comparison and tolerance as the
other product tests (the FP64 oracle, FP32 accumulation bound)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_15682_amd import reqat
from tests.test_gpu_parity import MX, NV, DEV, _rand, log, run_gemm_case

pytestmark = pytest.mark.gpu

# (tile, formats, M, N, K): the dispatch picks the named tile (asserted by the CPU test of its rules)
CASES = [
    ("64x128", (NV,), 65, 66, 128),             # half a stage
    ("64x128 deep", (MX,), 65, 66, 128),
    ("64x64", (NV, MX), 127, 65, 640),
    ("64x64", (NV, MX), 129, 130, 2176),        # five stages, K ends a quarter into the last
    ("64x64", (NV, MX), 193, 300, 4096),        # eight whole stages
    ("64x128", (NV,), 130, 12000, 384),
    ("64x128 deep", (MX,), 320, 6500, 384),
    ("64x128 deep", (NV,), 129, 10100, 2176),   # nine stages of 256
    ("128x128 deep", (MX,), 257, 8200, 640),
    ("128x128 deep", (MX,), 257, 8200, 1920),
    ("128x128", (NV,), 256, 32700, 128),
    ("64x128", (NV,), 1030, 16500, 1152),
    ("256x256", (NV, MX), 8100, 4000, 512),     # two tiles per workgroup
]


@pytest.mark.parametrize("fmt,M,N,K", [(f, M, N, K) for _, fmts, M, N, K in CASES for f in fmts])
def test_tile_kernels(fmt, M, N, K):
    log("gemm tiles fmt=%d M=%d N=%d K=%d" % (fmt, M, N, K))
    run_gemm_case(fmt, M, N, K, seed=M + N + K, dist="student_t", all_points=M * N <= 60000)


@pytest.mark.parametrize("fmt", [NV, MX])
@pytest.mark.parametrize("pad", [1, 4])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_of_y_keep_their_padding(fmt, pad, dtype):
    """y as a column slice, its rows 1 element (no vector store) or 4 past N: the same
    values as a dense y, and nothing written between the rows."""
    M, N, K = 70, 133, 640
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    ac, as_, ga = oracle.quantize(fmt, _rand(M, K, 1))
    bc, bs, gb = oracle.quantize(fmt, _rand(N, K, 2, std=0.02))
    gs = [None if fmt == MX else torch.tensor([g], dtype=torch.float32, device=DEV) for g in (ga, gb)]
    dense = reqat.gemm(fmt, t(ac), t(as_), gs[0], t(bc), t(bs), gs[1], out_dtype=dtype)
    wide = torch.full((M, N + pad), 7.0, dtype=dtype, device=DEV)
    reqat.gemm(fmt, t(ac), t(as_), gs[0], t(bc), t(bs), gs[1], out_dtype=dtype, out=wide[:, :N])
    torch.cuda.synchronize()
    assert torch.equal(wide[:, :N], dense) and bool((wide[:, N:] == 7.0).all())
