"""The large-block bf16 GEMM (csrc/prefill_gemm.hip): every tile instance on its own, at the edges of its
tiles (rows, columns and contraction steps that do not fill them, a split contraction) and through each
epilogue, against float64 products of the same bf16 operands.  The instances are called by their internal
launcher, since the shapes that select the largest of them are model-sized."""
import ctypes

import pytest
import torch

from paper_2403_18647_amd import binding as B

pytestmark = pytest.mark.gpu
STORE, QKV, SWIGLU = 0, 1, 2
TILES = [(16, 16), (16, 12), (16, 8), (16, 6), (8, 8), (8, 6), (8, 4), (8, 3)]   # kMma: 16-row, 16-column tiles


class Args(ctypes.Structure):   # PrefillGemmArgs (csrc/kernels.h)
    _p, _i = ctypes.c_void_p, ctypes.c_int
    _fields_ = [("M", _i), ("N", _i), ("K", _i), ("A", _p), ("lda", _i), ("W0", _p), ("W1", _p), ("W2", _p),
                ("n_per", _i), ("Wp", _p), ("n_tiles", _i), ("k_steps", _i), ("C", _p), ("ldc", _i), ("ksplit", _i),
                ("c_part", ctypes.c_size_t), ("ep", _i), ("q", _i), ("H", _i), ("Dh", _i), ("S_max", _i),
                ("cache_len", _p), ("rope", _p), ("qbuf", _p), ("kc", _p), ("vc", _p), ("err", _p), ("u", _p),
                ("ldu", _i)]


def _launch(cfg, a):
    L = B.lib()
    assert L._ZN5sdsat19prefill_mma_configsEv() == len(TILES)
    fn = L._ZN5sdsat18launch_prefill_mmaEiRKNS_15PrefillGemmArgsEP12ihipStream_t
    fn.argtypes = [ctypes.c_int, ctypes.POINTER(Args), ctypes.c_void_p]
    assert fn(cfg, ctypes.byref(a), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()


def _frag(x):
    """Rows [n, K] in fragment order, padded with zeros to whole 16-row tiles and 32-wide steps."""
    n, k = x.shape
    out = torch.zeros(((n + 15) // 16 * 16, (k + 31) // 32 * 32), dtype=x.dtype, device=x.device)
    out[:n, :k] = x
    return out.view(-1, 16, out.shape[1] // 8, 8).permute(0, 2, 1, 3).contiguous()


def _operands(m, n, k, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return [torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16) for s in ((m, k), (n, k))]


def _base(x, rows, wp, n, k, ep):
    a = Args()
    a.M, a.N, a.K, a.A, a.lda = rows, n, k, x.data_ptr(), (k + 31) // 32 * 32
    a.W0 = a.W1 = a.W2 = a.Wp = wp.data_ptr()
    a.n_per, a.n_tiles, a.k_steps, a.ksplit, a.ep = n, wp.shape[0], a.lda // 32, 1, ep
    return a


# one row past a row tile, a ragged last tile, exactly one tile; K: one step, fewer steps than stages in
# flight, an odd count, a ragged last step
@pytest.mark.parametrize("cfg", range(len(TILES)))
@pytest.mark.parametrize("k,ksplit", [(32, 1), (88, 1), (352, 1), (1056, 2)])
def test_store(cfg, k, ksplit):
    bm, bn = TILES[cfg]
    for m, n in ((16 * bm, 16 * bn), (16 * bm + 1, 16 * bn + 7), (70, 16), (16 * bm * 9 - 5, 16 * bn * 2 - 20)):
        x, w = _operands(m, n, k, 7 * m + k)
        xp, wp = _frag(x), _frag(w)
        c = torch.full((ksplit, m, n), 7e7, device="cuda")
        a = _base(xp, m, wp, n, k, STORE)
        a.C, a.ldc, a.ksplit, a.c_part = c.data_ptr(), n, ksplit, m * n
        _launch(cfg, a)
        ref = x.double() @ w.double().t()
        # float sums of k exact products: each of k + 1 additions rounds by at most 2^-24 of the running sum
        bound = (x.double().abs() @ w.double().abs().t()) * (k + 8) * 2.0 ** -24
        assert ((c.double().sum(0) - ref).abs() <= bound).all(), (cfg, m, n, k)


@pytest.mark.parametrize("cfg", range(len(TILES)))
@pytest.mark.parametrize("batch,q,dh,lens", [(1, 129, 128, [0]), (3, 67, 64, [5, 0, 30]), (2, 135, 128, [33, 2])])
def test_qkv(cfg, batch, q, dh, lens):
    """RoPE, the Q rows and the K / V slots, with sequence boundaries inside row tiles and cache lengths that
    leave the 4-key groups of V unaligned; slots of no row stay untouched."""
    h, k, s_max = 2, 96, 256
    d, m = h * dh, batch * q
    x, w = _operands(m, 3 * d, k, 11 + q)
    tph, half = dh // 16, dh // 2
    t = torch.arange(3 * d // 16)
    c = torch.arange(16)
    dim = 8 * (t % tph)[:, None] + torch.where(c < 8, c, half + c - 8)
    perm = ((t // tph * dh)[:, None] + dim).view(-1)
    xp, wp = _frag(x), _frag(w[perm.cuda()])
    ln = torch.tensor(lens, dtype=torch.int32, device="cuda")
    ang = torch.arange(s_max, dtype=torch.float64)[:, None] * 1e4 ** (-2.0 * torch.arange(half).double() / dh)
    rope = torch.stack([ang.cos(), ang.sin()], -1).float().cuda()
    qb = torch.full((m, h, dh), 7e7, device="cuda")
    kc = torch.full((batch, h, s_max, dh), 7.0, device="cuda", dtype=torch.bfloat16)
    vc = torch.full((batch, h, s_max // 32, dh, 32), 7.0, device="cuda", dtype=torch.bfloat16)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    a = _base(xp, m, wp, 3 * d, k, QKV)
    a.n_per, a.q, a.H, a.Dh, a.S_max = d, q, h, dh, s_max
    a.cache_len, a.rope, a.qbuf, a.kc, a.vc, a.err = (z.data_ptr() for z in (ln, rope, qb, kc, vc, err))
    _launch(cfg, a)
    y = (x.double() @ w.double().t()).view(batch, q, 3, h, dh)
    pos = (ln.long()[:, None] + torch.arange(q, device="cuda"))
    cs, sn = (rope.double()[pos][..., i][:, :, None, :] for i in (0, 1))

    def rot(z):
        lo, hi = z[..., :half], z[..., half:]
        return torch.cat([lo * cs - hi * sn, lo * sn + hi * cs], -1)

    tol = 1e-4   # 96 products of N(0,1) values: sums of about 10, float rounding of them 1e-6 each
    assert (qb.view(batch, q, h, dh).double() - rot(y[:, :, 0])).abs().max() < tol
    kb = torch.arange(32)
    vp = torch.where(kb < 16, kb // 4 * 8 + kb % 4, (kb - 16) // 4 * 8 + 4 + (kb - 16) % 4).cuda()
    v = vc[..., vp].permute(0, 1, 2, 4, 3).reshape(batch, h, s_max, dh)
    for got, ref in ((kc, rot(y[:, :, 1])), (v, y[:, :, 2])):
        want = torch.full((batch, h, s_max, dh), 7.0, dtype=torch.float64, device="cuda")
        for b in range(batch):
            want[b, :, lens[b]:lens[b] + q] = ref[b].transpose(0, 1)
        # one bf16 rounding (2^-9 of the value), or the neighbouring value where the float sum crossed a tie
        assert ((got.double() - want).abs() <= want.abs() * 2.0 ** -8 + tol).all(), cfg
    assert int(err) == 0


@pytest.mark.parametrize("cfg", range(len(TILES)))
@pytest.mark.parametrize("m,f", [(129, 688), (70, 40), (300, 1000)])
def test_swiglu(cfg, m, f):
    """silu(gate) * up in fragment order; the columns up to the padded length are zero whatever was there."""
    k, fp = 64, (f + 31) // 32 * 32
    x, w = _operands(m, 2 * f, k, f)
    t = torch.arange((f + 7) // 8)[:, None]
    c = torch.arange(16)
    row = 8 * t + c % 8
    wz = torch.cat([w, torch.zeros((1, k), device="cuda", dtype=torch.bfloat16)])
    perm = torch.where(row < f, torch.where(c < 8, row, f + row), torch.full_like(row, 2 * f)).view(-1)
    xp, wp = _frag(x), _frag(wz[perm.cuda()])
    u = torch.full(((m + 15) // 16, fp // 8, 16, 8), 7.0, device="cuda", dtype=torch.bfloat16)
    a = _base(xp, m, wp, 2 * f, k, SWIGLU)
    a.n_per, a.u, a.ldu = f, u.data_ptr(), fp
    _launch(cfg, a)
    y = x.double() @ w.double().t()
    want = torch.zeros((m, fp), dtype=torch.float64, device="cuda")
    want[:, :f] = y[:, :f] * torch.sigmoid(y[:, :f]) * y[:, f:]
    got = u.permute(0, 2, 1, 3).reshape(-1, fp)[:m].double()
    assert ((got - want).abs() <= want.abs() * 2.0 ** -8 + 1e-4).all(), cfg


def test_plan_is_an_instance():
    L = B.lib()
    for m in (65, 127, 128, 129, 511, 1023, 4092, 16384):
        for n_tiles in (16, 43, 256, 768, 1376, 2001):
            for split in (1, 2, 4):
                assert 0 <= L._ZN5sdsat16plan_prefill_mmaEiiii(m, n_tiles, 128, split) < len(TILES)
