"""GPU parity of the W4A4 product for rows of more than 2^26 elements, beyond the 32-bit
offsets of the tiles: the general kernel (more than 64 rows of X, its K loop and both edges of
its tile) and the skinny one.  Against the product of the exactly dequantized operands,
summed in 64 bits with torch, within the tolerance of the other product tests."""
import pytest
import torch

from paper_2606_15682_amd import reqat
from tests.test_gpu_parity import DEV, GEMM_TOL, MX, NV, log

pytestmark = pytest.mark.gpu

E2M1 = [0, 0.5, 1, 1.5, 2, 3, 4, 6]


def _dequantized(fmt, codes, scales):
    """float64 values of a run of columns (scale bytes of ordinary exponents)."""
    grid = torch.tensor(E2M1 + [-v for v in E2M1], dtype=torch.float64, device=DEV)
    v = grid[torch.stack([codes & 15, codes >> 4], -1).reshape(codes.shape[0], -1).int()]
    s = scales.int()
    s = torch.exp2((s - 127).double()) if fmt == MX else (1 + (s & 7) / 8).double() * torch.exp2(((s >> 3) - 7).double())
    B = reqat.BLOCK[fmt]
    return (v.reshape(len(v), -1, B) * s[:, :, None]).reshape(len(v), -1)


@pytest.mark.parametrize("fmt", [NV, MX])
def test_rows_beyond_2_to_the_26(fmt):
    M, N, K, B = 65, 130, (1 << 26) + 128, reqat.BLOCK[fmt]
    log("long rows fmt=%d M=%d N=%d K=%d" % (fmt, M, N, K))
    g = torch.Generator(device=DEV).manual_seed(7 + fmt)
    lo, hi = (120, 130) if fmt == MX else (0x30, 0x48)

    def operand(rows):
        return (torch.randint(0, 256, (rows, K // 2), generator=g, device=DEV, dtype=torch.uint8),
                torch.randint(lo, hi, (rows, K // B), generator=g, device=DEV, dtype=torch.uint8))

    ac, as_ = operand(M)
    bc, bs = operand(N)
    one = None if fmt == MX else torch.tensor([0.5], dtype=torch.float32, device=DEV)
    y = reqat.gemm(fmt, ac, as_, one, bc, bs, one)
    few = reqat.gemm(fmt, ac[:20], as_[:20], one, bc, bs, one)
    torch.cuda.synchronize()
    log("products done")
    ref = torch.zeros((M, N), dtype=torch.float64, device=DEV)
    mag = torch.zeros_like(ref)
    step = 1 << 20
    for k in range(0, K, step):
        a, b = (_dequantized(fmt, c[:, k // 2:(k + step) // 2], s[:, k // B:(k + step) // B])
                for c, s in ((ac, as_), (bc, bs)))
        ref += torch.mm(a, b.t().contiguous())
        mag += torch.mm(a.abs(), b.abs().t().contiguous())
    scale = 1.0 if fmt == MX else 0.25
    for got, rows in ((y, M), (few, 20)):
        assert bool(((got.double() - scale * ref[:rows]).abs() <= GEMM_TOL * scale * mag[:rows]).all())
        # the sums are far smaller than the sum of magnitudes: the result itself is right too
        assert float((got.double() - scale * ref[:rows]).norm() / (scale * ref[:rows]).norm()) < 0.05
