"""Skinny GEMMs of several row tiles on wide matrices (three column tiles per workgroup): row and column
remainders, a ragged contraction, and each row bit for bit as in a one-row product."""
import pytest
import torch

from paper_2403_18647_amd import binding as B

pytestmark = pytest.mark.gpu


def _linear(m, n, k, x, packed):
    y = torch.full((m, n), 7e7, device="cuda")
    scratch = torch.empty(B.sdsat_linear_scratch_bytes(m, n, k), dtype=torch.uint8, device="cuda")
    B.sdsat_linear(B.DTYPE_BF16, m, n, k, x, packed, y, scratch)
    torch.cuda.synchronize()
    return y


@pytest.mark.parametrize("m", [17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("n,k", [(513 * 16 + 5, 200), (515 * 16, 544)])   # 1 and 2 tiles past whole groups
def test_three_tiles(m, n, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(m + k)
    x = torch.randn((m, k), generator=g, device="cuda")
    w = torch.randn((n, k), generator=g, device="cuda", dtype=torch.bfloat16)
    packed = torch.empty(B.sdsat_linear_packed_bytes(B.DTYPE_BF16, n, k), dtype=torch.uint8, device="cuda")
    B.sdsat_linear_pack(B.DTYPE_BF16, n, k, w, packed)
    y = _linear(m, n, k, x, packed)
    xb = x.bfloat16().double()
    # float sums of k exact products: k + 8 additions, each off by at most 2^-24 of the running sum
    bound = (xb.abs() @ w.double().abs().t()) * (k + 8) * 2.0 ** -24
    assert ((y.double() - xb @ w.double().t()).abs() <= bound).all()
    for r in (0, 16, m - 1):
        assert torch.equal(_linear(1, n, k, x[r:r + 1].contiguous(), packed)[0], y[r]), r
