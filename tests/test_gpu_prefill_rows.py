"""Rows of a large block (more than 64 rows) against the kernels of decode blocks, bit for bit: layer 0's
normalised rows, RoPE's rounding, and attention rows whose keys lie in one 32-key block.  A token then enters
layer 0 the same whether it comes in a prompt or in a draft block."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2403_18647_amd import binding as B
from paper_2403_18647_amd import synth
from test_gpu_prefill_mma import QKV, STORE, _base, _frag, _launch, _operands

pytestmark = pytest.mark.gpu


def _unfrag(h, m, d):
    """Rows in fragment order whose last 16-row tile holds only its real rows, as [m, d]."""
    out = torch.empty((m, d), dtype=h.dtype, device=h.device)
    for t in range(0, m, 16):
        r = min(16, m - t)
        out[t:t + r] = h[t * d:(t + r) * d].view(d // 8, r, 8).transpose(0, 1).reshape(r, d)
    return out


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("m,d", [(65, 64), (127, 256), (70, 1088), (66, 8192)])
def test_layer0_rows(dtype, m, d):
    """The one-pass embedding and RMSNorm of a large block, and the decode block's two kernels."""
    L = B.lib()
    one = L._ZN5sdsat22launch_embed_norm_rowsEiPKviPKiiiPfPKffPviPiP12ihipStream_t
    emb = L._ZN5sdsat12launch_embedEiPKviiPKiiPfS4_PKfiS4_iPiP12ihipStream_t
    rms = L._ZN5sdsat15launch_rms_rowsEiPKfiS1_iifiPvP12ihipStream_t
    P, I, F = ctypes.c_void_p, ctypes.c_int, ctypes.c_float
    one.argtypes = [I, P, I, P, I, I, P, P, F, P, I, P, P]
    emb.argtypes = [I, P, I, I, P, I, P, P, P, I, P, I, P, P]
    rms.argtypes = [I, P, I, P, I, I, F, I, P, P]
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    t = torch.bfloat16 if dtype else torch.float32
    e = torch.randn((50, d), generator=g, device="cuda").to(t)
    gain = 1 + 0.1 * torch.randn(d, generator=g, device="cuda")
    tok = torch.randint(0, 50, (m,), generator=g, device="cuda", dtype=torch.int32)
    m16, n_ssq = (m + 15) // 16 * 16, d // 16
    x, x1, xg = (torch.zeros((m16, d), device="cuda") for _ in range(3))
    ssq = torch.zeros((m, n_ssq), device="cuda")
    h, h1 = (torch.zeros(m16 * d, device="cuda", dtype=t) for _ in range(2))
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    p = [z.data_ptr() for z in (e, tok, x, gain, h, err, x1, xg, ssq, h1)]
    assert one(dtype, p[0], 50, p[1], m, d, p[2], p[3], 1e-5, p[4], d, p[5], st) == 0
    assert emb(dtype, p[0], 50, d, p[1], m, p[6], p[7], p[3], d, p[8], n_ssq, p[5], st) == 0
    assert rms(dtype, p[7], d, p[8], n_ssq, d, 1e-5, m, p[9], st) == 0
    torch.cuda.synchronize()
    assert torch.equal(x, x1) and int(err) == 0
    # the large block keeps whole 16-row tiles
    got = h.view(m16 // 16, d // 8, 16, 8).transpose(1, 2).reshape(m16, d)[:m]
    assert torch.equal(got, _unfrag(h1, m, d))


@pytest.mark.parametrize("cfg", [0, 4, 7])
def test_rope_rounding(cfg):
    """Q and K of the QKV epilogue from the same GEMM's plain output: y1 = x1 cos - round(x2 sin) and
    y2 = x2 cos + round(x1 sin), each one fused multiply-add."""
    h, dh, k, m, s_max = 2, 128, 96, 129, 256
    d, half = h * dh, dh // 2
    x, w = _operands(m, 3 * d, k, 3)
    t, c = torch.arange(3 * d // 16), torch.arange(16)
    dim = 8 * (t % (dh // 16))[:, None] + torch.where(c < 8, c, half + c - 8)
    perm = ((t // (dh // 16) * dh)[:, None] + dim).view(-1).cuda()
    xp, wp, wq = _frag(x), _frag(w[perm]), _frag(w)
    y = torch.empty((m, 3 * d), device="cuda")
    a = _base(xp, m, wq, 3 * d, k, STORE)
    a.C, a.ldc, a.c_part = y.data_ptr(), 3 * d, m * 3 * d
    _launch(cfg, a)
    rope = torch.randn((s_max, half, 2), device="cuda")   # any table
    ln = torch.zeros(1, dtype=torch.int32, device="cuda")
    qb = torch.empty((m, h, dh), device="cuda")
    kc = torch.zeros((h, s_max, dh), device="cuda", dtype=torch.bfloat16)
    vc = torch.zeros((h, s_max, dh), device="cuda", dtype=torch.bfloat16)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    a = _base(xp, m, wp, 3 * d, k, QKV)
    a.n_per, a.q, a.H, a.Dh, a.S_max = d, m, h, dh, s_max
    a.cache_len, a.rope, a.qbuf, a.kc, a.vc, a.err = (z.data_ptr() for z in (ln, rope, qb, kc, vc, err))
    _launch(cfg, a)
    v = y.view(m, 3, h, dh).cpu().numpy()
    cs, sn = (rope[:m, None, :, i].cpu().numpy() for i in (0, 1))

    def fma(a, b, c):   # a b is exact in 64 bits; their sum with c rounds once more there, at 2^-53 of it
        return (a.astype(np.float64) * b + c).astype(np.float32)

    def rot(z):
        lo, hi = z[..., :half], z[..., half:]
        return torch.from_numpy(np.concatenate([fma(lo, cs, -(hi * sn)), fma(hi, cs, lo * sn)], -1))

    assert torch.equal(qb.cpu(), rot(v[:, 0]))
    assert torch.equal(kc[:, :m].cpu(), rot(v[:, 1]).transpose(0, 1).bfloat16())


@pytest.mark.parametrize("dh,heads,batch", [(128, 2, 1), (64, 4, 1), (128, 2, 65), (64, 2, 65)])   # both workgroup sizes
def test_attention_one_key_block(dh, heads, batch):
    sh = synth.small_shape(n_layers=1, d_model=heads * dh, n_heads=heads, head_dim=dh, d_ffn=64, vocab=64, dtype="bf16")
    g = torch.Generator(device="cuda")
    g.manual_seed(dh)
    w = [torch.zeros(synth.tensor_shape(sh, n), device="cuda", dtype=torch.float32 if synth.is_gain(n) else torch.bfloat16)
         for n in synth.tensor_names(sh)]
    kv = [torch.randn((batch, 96, heads, dh), generator=g, device="cuda") for _ in range(2)]
    pos = torch.arange(96, dtype=torch.int32, device="cuda").repeat(batch)
    qs = torch.randn((batch, 65, heads * dh), generator=g, device="cuda") * 2
    outs = []
    for q in (65, 26):
        ctx = B.Context(B.make_config(sh, batch, 96, 65), w)
        B.sdsat_kv_write(ctx.handle, 0, batch, 96, *kv, pos)
        B.sdsat_set_cache_len(ctx.handle, [5] * batch)
        out = torch.empty((batch, q, heads * dh), device="cuda")
        B.sdsat_attention(ctx.handle, 0, batch, q, qs[:, :q].contiguous(), None, out)
        torch.cuda.synchronize()
        outs.append(out[:, :26])
        ctx.close()
    assert torch.equal(*outs)
