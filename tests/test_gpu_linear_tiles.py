"""Skinny GEMMs of several row tiles on wide matrices (three column tiles per workgroup): row and column
remainders, a ragged contraction, and each row bit for bit as in a one-row product."""
import pytest
import torch

from paper_2403_18647_amd import binding as B
from paper_2403_18647_amd import synth

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


@pytest.mark.parametrize("batch", [3, 5, 8])   # 2, 3 and 4 row tiles
def test_residual_beyond_512_tiles(batch):
    """d_model > 8192: the O and down GEMMs of blocks of 17 to 64 rows, whole (not split), give each sequence the
    values of its own 8-row block."""
    sh = synth.small_shape(n_layers=1, d_model=8320, n_heads=65, head_dim=128, d_ffn=256, vocab=64, dtype="bf16")
    g = torch.Generator(device="cuda")
    g.manual_seed(batch)
    w = [1 + 0.1 * torch.randn(synth.tensor_shape(sh, n), generator=g, device="cuda") if synth.is_gain(n) else
         0.02 * torch.randn(synth.tensor_shape(sh, n), generator=g, device="cuda", dtype=torch.bfloat16)
         for n in synth.tensor_names(sh)]
    tok = torch.randint(0, 64, (batch, 8), generator=g, device="cuda", dtype=torch.int32)
    ctx = B.Context(B.make_config(sh, batch, 32, 8), w)
    out = torch.empty((batch, 8, 64), device="cuda")
    one = torch.empty_like(out)
    B.sdsat_forward_block(ctx.handle, batch, 8, tok, None, out)
    for b in range(batch):
        B.sdsat_forward_block(ctx.handle, 1, 8, tok[b:b + 1].contiguous(), None, one[b])
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(out, one)
