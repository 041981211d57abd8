"""Prefill attention of bf16 models (blocks of more than 64 rows) at the edges of its 64-row tiles, 32-row
waves, key-block steps and workgroup widths (up to 256 tiles, more), against float64 softmax attention over
the same bf16 keys and values."""
import math

import pytest
import torch

from paper_2403_18647_amd import binding as B
from paper_2403_18647_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh,heads,batch,q,lens", [
    (128, 2, 1, 65, [0]), (64, 4, 1, 65, [0]),            # a second tile of one row, no cache
    (128, 2, 2, 96, [31, 1]), (64, 4, 2, 97, [32, 129]),  # half a tile; one row past half, ragged caches
    (128, 2, 1, 128, [640]), (64, 4, 1, 200, [1000]),     # many steps before the diagonal
    (128, 32, 3, 190, [3, 0, 77]), (64, 64, 2, 131, [5, 96]),   # more than 256 tiles: the narrow workgroups
])
def test_against_float64(dh, heads, batch, q, lens):
    sh = synth.small_shape(n_layers=1, d_model=heads * dh, n_heads=heads, head_dim=dh, d_ffn=64, vocab=64, dtype="bf16")
    w = [torch.zeros(synth.tensor_shape(sh, n), device="cuda", dtype=torch.float32 if synth.is_gain(n) else torch.bfloat16)
         for n in synth.tensor_names(sh)]
    n = max(lens) + q
    ctx = B.Context(B.make_config(sh, batch, n, q), w)
    g = torch.Generator(device="cuda")
    g.manual_seed(q)
    k, v = (torch.randn((batch, n, heads, dh), generator=g, device="cuda").bfloat16().float() for _ in range(2))
    pos = torch.arange(n, dtype=torch.int32, device="cuda").repeat(batch)
    B.sdsat_kv_write(ctx.handle, 0, batch, n, k, v, pos)
    B.sdsat_set_cache_len(ctx.handle, lens)
    qs = torch.randn((batch * q, heads * dh), generator=g, device="cuda") * 2
    out = torch.full((batch * q, heads * dh), 7e7, device="cuda")
    B.sdsat_attention(ctx.handle, 0, batch, q, qs, None, out)
    torch.cuda.synchronize()
    for b, ln in enumerate(lens):
        t = ln + q
        kb, vb = (z[b, :t].double().transpose(0, 1).contiguous() for z in (k, v))
        qb = qs.view(batch, q, heads, dh)[b].double().transpose(0, 1).contiguous()
        s = torch.matmul(qb, kb.transpose(1, 2).contiguous()) / math.sqrt(dh)
        see = torch.ones((q, t), dtype=torch.bool, device="cuda").tril(ln)
        ref = torch.matmul(s.masked_fill(~see, -math.inf).softmax(-1), vb).transpose(0, 1).reshape(q, -1)
        got = out.view(batch, q, -1)[b].double()
        # scores and probabilities enter the matrix cores with about 16 significant bits (value + remainder):
        # scores of |s| <= 2 sqrt(dh) * 4 err by 2^-17 of their terms' size, which moves an output by that factor
        assert float((got - ref).abs().max()) < 1e-3, (b, float((got - ref).abs().max()))
    ctx.close()
