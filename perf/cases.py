"""Performance cases: the work a user of this library has it do, through the entry points of include/sdsat.h.

Five kinds of call, each over the range its users meet:

* ``block``     one draft or verify block of the decode loop: sdsat_forward_block over batch x q rows against
                a filled KV cache, logits of every row out (chain or draft-tree mask);
* ``prefill``   the prompt: sdsat_reset, sdsat_forward_block without logits, sdsat_commit_kv, then the first
                draft block with its logits (what a program waits for before its first token);
* ``attention`` sdsat_attention over a long cache;
* ``greedy`` / ``nucleus``  sdsat_verify_greedy / sdsat_verify_nucleus on logits, drafts given.

Models have the widths, head sizes, vocabularies and slot counts of the 7B, 13B and tiny decoders in
paper_2403_18647_amd/synth.py and a few of their layers: every layer costs the same, a few already exceed the
caches, and a rounding difference does not travel through 32 layers.  Weights are N(0, 0.02), cached K and V
N(0, 1), logits N(0, 4).
"""
import math

import numpy as np
import torch

from paper_2403_18647_amd import binding as B
from paper_2403_18647_amd import synth

MODELS = {"tiny": synth.TINY, "7b": synth.LLAMA7B, "13b": synth.LLAMA13B,
          # the reduced bf16 decoder of the tests: 128-wide heads, ragged vocabulary and FFN tiles
          "small": synth.small_shape(n_layers=2, d_model=256, n_heads=2, head_dim=128, d_ffn=688, vocab=1000,
                                     n_adaptive=5, rope_base=1e6, dtype="bf16")}


def listed():
    return [
        # the tiny fp32 decoder's draft block: a couple of megabytes of weights, so launches and latency
        {"name": "tiny_block", "kind": "block", "model": "tiny", "layers": 2, "batch": 1, "q": 6, "ctx": 64,
         "slots": 128, "tree": 0},
        # verification of a batch-1 greedy loop, k = 5: one of the many small calls between two blocks
        {"name": "greedy_b1", "kind": "greedy", "batch": 1, "q": 6, "vocab": 32016},
        # verification of the batch-4 nucleus loop (top-p 0.95, T 0.8)
        {"name": "nucleus_b4", "kind": "nucleus", "batch": 4, "q": 6, "vocab": 32016, "T": 0.8, "p": 0.95, "k": 0},
        # the decode block of the 7B greedy workload: batch 1, k = 5, 512-token prompt plus half the new tokens
        {"name": "7b_b1_q6", "kind": "block", "model": "7b", "layers": 4, "batch": 1, "q": 6, "ctx": 640,
         "slots": 832, "tree": 0},
        # the decode block of the 13B workload: k = 10, 2048-token prompt
        {"name": "13b_b1_q11", "kind": "block", "model": "13b", "layers": 3, "batch": 1, "q": 11, "ctx": 2303,
         "slots": 2592, "tree": 0},
        # the decode block of the batch-4 workload (1024-token prompts, ragged lengths)
        {"name": "7b_b4_q6", "kind": "block", "model": "7b", "layers": 4, "batch": 4, "q": 6, "ctx": 1150,
         "slots": 1312, "tree": 0},
        # draft step 2 of the tree loop at batch 4: width 2, k = 5, ancestor masks
        {"name": "7b_b4_tree11", "kind": "block", "model": "7b", "layers": 4, "batch": 4, "q": 11, "ctx": 1150,
         "slots": 1312, "tree": 2},
        # a serving program's own loop at batch 8, k = 10: more rows than the skinny GEMMs take
        {"name": "7b_b8_q11", "kind": "block", "model": "7b", "layers": 4, "batch": 8, "q": 11, "ctx": 600,
         "slots": 832, "tree": 0},
        # a short prompt (a function signature with its docstring)
        {"name": "7b_prefill_127", "kind": "prefill", "model": "7b", "layers": 4, "batch": 1, "rows": 127, "q": 6},
        # the 512-token prompt of the 7B workload
        {"name": "7b_prefill_511", "kind": "prefill", "model": "7b", "layers": 4, "batch": 1, "rows": 511, "q": 6},
        # the four 1024-token prompts of the batch-4 workload
        {"name": "7b_prefill_4x1023", "kind": "prefill", "model": "7b", "layers": 2, "batch": 4, "rows": 1023, "q": 6},
        # attention of a long-context batch: 8 sequences of 16384 cached keys, k = 5
        {"name": "attention_16k", "kind": "attention", "batch": 8, "q": 6, "ctx": 16384, "heads": 32, "head_dim": 128},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["block", "block", "block", "block", "prefill", "prefill", "prefill", "attention", "greedy",
                       "nucleus"])
    if kind == "block":
        model = rng.choice(["7b", "7b", "7b", "13b", "tiny", "small"])
        if rng.random() < 0.25:
            # past the skinny GEMMs' 64 rows
            batch = rng.randint(5, 16)
            q, tree = rng.randint(64 // batch + 1, 16), 0
        else:
            batch = _log_int(rng, 1, 10)
            q = rng.randint(1, min(14, 64 // batch))
            tree = 2 if q >= 3 and q % 2 == 1 and rng.random() < 0.4 else 0
        ctx = _log_int(rng, 16, 4096 if batch <= 2 else 1500)
        return {"kind": "block", "model": model, "layers": rng.randint(2, 4), "batch": batch, "q": q, "ctx": ctx,
                "slots": ctx + q + rng.randint(0, 400), "tree": tree}
    if kind == "prefill":
        model = rng.choice(["7b", "7b", "7b", "13b", "small", "tiny"])
        batch = _log_int(rng, 1, 4)
        layers = 2
        most = 4000 // batch if model != "13b" else 2500 // batch
        return {"kind": "prefill", "model": model, "layers": layers, "batch": batch,
                "rows": _log_int(rng, 20, min(2047, most)), "q": rng.randint(1, 11)}
    if kind == "attention":
        ctx = _log_int(rng, 64, 16384)
        heads, dh = rng.choice([(32, 128), (40, 128), (4, 64)])
        return {"kind": "attention", "batch": rng.randint(1, 8), "q": rng.randint(1, 16), "ctx": ctx, "heads": heads,
                "head_dim": dh}
    batch, q = rng.randint(1, 8), rng.randint(1, 11)
    vocab = rng.choice([1000, 1024, 32000, 32016, 32016, 32016, 128256])
    if kind == "greedy":
        return {"kind": "greedy", "batch": batch, "q": q, "vocab": vocab}
    return {"kind": "nucleus", "batch": batch, "q": q, "vocab": vocab, "T": rng.choice([0.2, 0.8, 1.0]),
            "p": rng.choice([0.9, 0.95, 1.0]), "k": rng.choice([0, 0, 10, 50, 500])}


# ------------------------------------------------------------------ inputs (from the seed alone)
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _model(case):
    return synth.replace(MODELS[case["model"]], n_layers=case["layers"])


def _weights(case, g):
    """The model's tensors in the library's order (matrices in the model's type, gains float32)."""
    sh = _model(case)
    dt = torch.bfloat16 if sh.dtype == "bf16" else torch.float32
    out = []
    for name in synth.tensor_names(sh):
        shape = synth.tensor_shape(sh, name)
        if synth.is_gain(name):
            out.append(1.0 + 0.1 * torch.randn(shape, generator=g, device="cuda"))
        else:
            out.append((torch.randn(shape, generator=g, device="cuda", dtype=dt)).mul_(0.02))
    return out


def _lens(case):
    """Committed tokens per sequence: ragged, the longest first."""
    return [max(1, case["ctx"] - 61 * b % max(1, case["ctx"])) for b in range(case["batch"])]


def _cache_kv(case, layers, heads, head_dim, bf16, g):
    """K and V of every layer and sequence as stored (float tensors of bf16 values for bf16 models)."""
    n = max(_lens(case))
    for _ in range(layers):
        kv = []
        for _ in range(2):
            t = torch.randn((case["batch"], n, heads, head_dim), generator=g, device="cuda")
            kv.append(t.bfloat16().float() if bf16 else t)
        yield kv


def _tree(q, width):
    """Depths and ancestor masks of a draft tree: root, the chain, then the other candidates of each depth as leaves."""
    k = (q - 1) // width
    depth, mask = [0], [1]
    for j in range(1, k + 1):
        depth.append(j)
        mask.append((1 << (j + 1)) - 1)
    for j in range(1, k + 1):
        for _ in range(width - 1):
            r = len(depth)
            depth.append(j)
            mask.append(((1 << j) - 1) | (1 << r))
    return depth, mask


def _tokens(sh, shape, g):
    """Ids of prompt or block rows (adaptive ids among them)."""
    return torch.randint(0, sh.vocab + sh.n_adaptive, shape, generator=g, device="cuda", dtype=torch.int32)


def _logits(case, g):
    return torch.randn((case["batch"] * case["q"], case["vocab"]), generator=g, device="cuda").mul_(4.0)


def _drafts(case, logits, g):
    """k drafts per sequence, the first b mod (k + 1) of them the arg-max of the row before."""
    k = case["q"] - 1
    d = torch.randint(0, case["vocab"], (case["batch"], max(k, 1)), generator=g, device="cuda", dtype=torch.int32)
    best = logits.argmax(-1).view(case["batch"], case["q"]).int()
    for b in range(case["batch"]):
        n = b % (k + 1)
        d[b, :n] = best[b, :n]
    return d


# ------------------------------------------------------------------ what a program holds before the call
def prepare(case, seed):
    g = _gen(seed)
    kind, batch, q = case["kind"], case["batch"], case["q"]
    if kind in ("greedy", "nucleus"):
        # a context of any model with this vocabulary serves (verification reads only the logits)
        sh = synth.small_shape(n_layers=1, vocab=case["vocab"])
        w = _weights_like(sh)
        ctx = B.Context(B.make_config(sh, batch, 32, max(q, 1)), w)
        logits = _logits(case, g)
        return {"case": case, "ctx": ctx, "logits": logits, "drafts": _drafts(case, logits, g),
                "pos0": torch.full((batch,), 700, dtype=torch.int32, device="cuda"), "seed": seed,
                "tokens": torch.empty((batch, q), dtype=torch.int32, device="cuda"),
                "accept": torch.empty(batch, dtype=torch.int32, device="cuda")}
    if kind == "attention":
        sh = synth.small_shape(n_layers=1, d_model=case["heads"] * case["head_dim"], n_heads=case["heads"],
                               head_dim=case["head_dim"], d_ffn=64, vocab=64, dtype="bf16")
        ctx = B.Context(B.make_config(sh, batch, case["ctx"] + q, q), _weights_like(sh))
        _fill_cache(ctx, case, 1, sh, g)
        return {"case": case, "ctx": ctx,
                "q": torch.randn((batch * q, sh.d_model), generator=g, device="cuda"),
                "out": torch.empty((batch * q, sh.d_model), device="cuda")}
    sh = _model(case)
    w = _weights(case, g)
    if kind == "block":
        ctx = B.Context(B.make_config(sh, batch, case["slots"], q), w)
        _fill_cache(ctx, case, sh.n_layers, sh, g)
        mask = None
        if case["tree"]:
            mask = torch.tensor(_tree(q, case["tree"])[1] * batch, dtype=torch.int64, device="cuda")
        return {"case": case, "ctx": ctx, "tokens": _tokens(sh, (batch, q), g), "mask": mask,
                "logits": torch.empty((batch * q, sh.vocab), device="cuda")}
    rows = case["rows"]
    ctx = B.Context(B.make_config(sh, batch, rows + 256 + 2 * q, max(rows, q)), w)
    return {"case": case, "ctx": ctx, "prompt": _tokens(sh, (batch, rows), g), "tokens": _tokens(sh, (batch, q), g),
            "n": torch.full((batch,), rows, dtype=torch.int32, device="cuda"),
            "logits": torch.empty((batch * q, sh.vocab), device="cuda")}


def _weights_like(sh):
    """Zero weights for calls that read none."""
    dt = torch.bfloat16 if sh.dtype == "bf16" else torch.float32
    return [torch.zeros(synth.tensor_shape(sh, n), device="cuda", dtype=torch.float32 if synth.is_gain(n) else dt)
            for n in synth.tensor_names(sh)]


def _fill_cache(ctx, case, layers, sh, g):
    lens = _lens(case)
    n = max(lens)
    pos = torch.arange(n, dtype=torch.int32, device="cuda").repeat(case["batch"])
    for layer, (k, v) in enumerate(_cache_kv(case, layers, sh.n_heads, sh.head_dim, sh.dtype == "bf16", g)):
        B.sdsat_kv_write(ctx.handle, layer, case["batch"], n, k, v, pos)
        torch.cuda.synchronize()   # k and v are freed here
    B.sdsat_set_cache_len(ctx.handle, lens)


# ------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    h, kind, batch, q = s["ctx"].handle, case["kind"], case["batch"], case["q"]
    if kind == "block":
        B.sdsat_forward_block(h, batch, q, s["tokens"], s["mask"], s["logits"])
        return s["logits"]
    if kind == "prefill":
        B.sdsat_reset(h, batch)
        B.sdsat_forward_block(h, batch, case["rows"], s["prompt"], None, None)
        B.sdsat_commit_kv(h, batch, case["rows"], s["n"])
        B.sdsat_forward_block(h, batch, q, s["tokens"], None, s["logits"])
        return s["logits"]
    if kind == "attention":
        B.sdsat_attention(h, 0, batch, q, s["q"], None, s["out"])
        return s["out"]
    drafts = s["drafts"] if q > 1 else None
    if kind == "greedy":
        B.sdsat_verify_greedy(h, batch, q, s["logits"], drafts, s["tokens"], s["accept"])
    else:
        B.sdsat_verify_nucleus(h, batch, q, s["logits"], drafts, case["T"], case["p"], case["k"], s["seed"],
                               s["pos0"], s["tokens"], s["accept"])
    return s["tokens"], s["accept"]


# ------------------------------------------------------------------ what a pass cannot do without
def _forward_work(sh, batch, q, lens, logits):
    """Bytes and operations of one block forward over lens[b] cached tokens per sequence."""
    e = 2 if sh.dtype == "bf16" else 4
    d, f, m = sh.d_model, sh.d_ffn, batch * q
    layer_w = 4 * d * d + 3 * d * f
    by = sh.n_layers * layer_w * e + (2 * sh.n_layers + 1) * d * 4 + m * (d * e + 4)
    fl = 2.0 * m * sh.n_layers * layer_w
    for n in lens:
        by += sh.n_layers * 2 * (n + q) * d * e              # cached keys and values read, the block's written
        fl += sh.n_layers * 4.0 * d * (q * n + q * (q + 1) / 2)
    if logits:
        by += sh.vocab * d * e + m * sh.vocab * 4
        fl += 2.0 * m * sh.vocab * d
    return by, fl


def work(case):
    kind, batch, q = case["kind"], case["batch"], case["q"]
    if kind == "block":
        by, fl = _forward_work(_model(case), batch, q, _lens(case), True)
    elif kind == "prefill":
        sh = _model(case)
        by, fl = _forward_work(sh, batch, case["rows"], [0] * batch, False)
        by2, fl2 = _forward_work(sh, batch, q, [case["rows"]] * batch, True)
        by, fl = by + by2, fl + fl2
    elif kind == "attention":
        d = case["heads"] * case["head_dim"]
        by = sum(2 * (n + q) * d * 2 for n in _lens(case)) + 2 * batch * q * d * 4
        fl = sum(4.0 * d * (q * n + q * (q + 1) / 2) for n in _lens(case))
    else:
        by = batch * q * case["vocab"] * 4 + batch * (q - 1) * 4 + batch * q * 4 + batch * 4
        fl = batch * q * case["vocab"] * (1.0 if kind == "greedy" else 4.0)
    return {"bytes": by, "flops": fl}


def tolerance(case):
    kind = case["kind"]
    if kind in ("greedy", "nucleus"):
        return "exact"
    if kind == "attention":
        # against 64 bits the output is 3.4e-6 off (largest 1.8e-5): Q and P as bf16 pairs, float sums
        return {"rel": 2e-5, "max": 2e-4}
    if MODELS[case["model"]].dtype == "fp32":
        # 4e-7 to 6e-7 off (largest 2.4e-6); float sums in another order
        return {"rel": 3e-6, "max": 2e-5}
    # 0.004 to 0.014 off (largest 0.07): a handful of bf16 storage roundings per layer; another summation order
    # flips some of them, and each flip changes what follows
    return {"rel": 2.5e-2, "max": 0.25}


# ------------------------------------------------------------------ the same in 64 bits
def _rope(x, pos, base):
    """x [rows, H, Dh] float64, rotate-half pairs (i, i + Dh / 2)."""
    half = x.shape[-1] // 2
    inv = base ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / x.shape[-1])
    ang = pos.double()[:, None] * inv
    cs, sn = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * cs - b * sn, a * sn + b * cs], -1)


def _attend(qh, k, v, see):
    """qh [q, H, Dh] over k, v [n, H, Dh], see [q, n] visible keys; all float64."""
    out = torch.empty_like(qh)
    for h0 in range(0, qh.shape[1], 8):   # a few heads at a time bounds the memory
        hs = slice(h0, h0 + 8)
        s = torch.matmul(qh[:, hs].transpose(0, 1).contiguous(), k[:, hs].permute(1, 2, 0).contiguous())
        s = (s / math.sqrt(qh.shape[-1])).masked_fill(~see, -math.inf)
        out[:, hs] = torch.matmul(s.softmax(-1), v[:, hs].transpose(0, 1).contiguous()).transpose(0, 1)
    return out


def _norm(x, gain, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _forward(sh, w, caches, tokens, mask, depth, logits):
    """Block forward of the whole batch in float64: caches[layer][b] = (k, v) float64 [n_b, H, Dh]; returns the
    logits (or None) and appends the block's keys and values to the caches."""
    batch, q = tokens.shape
    dev = tokens.device
    x = w[0][tokens.reshape(-1).long()].double()
    tri = torch.ones((q, q), dtype=torch.bool, device=dev).tril()
    if mask is not None:
        tri = torch.tensor([[(mask[r] >> j) & 1 for j in range(q)] for r in range(q)], device=dev).bool()
    dep = torch.tensor(depth if depth is not None else list(range(q)), device=dev)
    for l in range(sh.n_layers):
        an, wq, wk, wv, wo, fn, wg, wu, wd = w[1 + 9 * l: 10 + 9 * l]
        h = _norm(x, an, sh.rms_eps)
        qq, kk, vv = ((h @ m.double().t()).view(batch, q, sh.n_heads, sh.head_dim) for m in (wq, wk, wv))
        o = torch.empty((batch, q, sh.n_heads, sh.head_dim), dtype=torch.float64, device=dev)
        for b in range(batch):
            k0, v0 = caches[l][b]
            pos = dep + k0.shape[0]
            k1 = torch.cat([k0, _rope(kk[b], pos, sh.rope_base)])
            v1 = torch.cat([v0, vv[b]])
            see = torch.cat([torch.ones((q, k0.shape[0]), dtype=torch.bool, device=dev), tri], 1)
            o[b] = _attend(_rope(qq[b], pos, sh.rope_base), k1, v1, see)
            caches[l][b] = (k1, v1)
        x = x + o.view(batch * q, -1) @ wo.double().t()
        h = _norm(x, fn, sh.rms_eps)
        gate = h @ wg.double().t()
        x = x + (gate * torch.sigmoid(gate) * (h @ wu.double().t())) @ wd.double().t()
    if not logits:
        return None
    return _norm(x, w[-2], sh.rms_eps) @ w[-1].double().t()


def _splitmix(state, n):
    m = (1 << 64) - 1
    z = (state + n * 0x9E3779B97F4A7C15) & m
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
    return z ^ (z >> 31)


def _sample(row, temp, p, k, u):
    """One row's nucleus draw: temperature, the top_k largest (ties keep lower ids), the smallest value threshold
    whose mass reaches p (every id tied at it kept), inverse CDF in ascending id order."""
    z = row.double() / temp
    e = (z - z.max()).exp()
    order = torch.sort(row, descending=True, stable=True)[1]
    if 0 < k < row.numel():
        order = order[:k]
    cum = e[order].cumsum(0)
    n = int((cum < min(1.0, p) * cum[-1]).sum())
    n = min(n, order.numel() - 1)
    keep = torch.zeros_like(row, dtype=torch.bool)
    keep[order] = True
    keep &= row >= row[order[n]]
    ids = keep.nonzero().view(-1)
    c = e[ids].cumsum(0)
    j = int((c <= u * c[-1]).sum())
    return int(ids[min(j, ids.numel() - 1)])


def exact(case, seed):
    g = _gen(seed)
    kind, batch, q = case["kind"], case["batch"], case["q"]
    if kind in ("greedy", "nucleus"):
        logits = _logits(case, g)
        drafts = _drafts(case, logits, g).cpu()
        if kind == "greedy":
            tok = logits.argmax(-1).view(batch, q).int().cpu()
        else:
            tok = torch.empty((batch, q), dtype=torch.int32)
            for b in range(batch):
                for j in range(q):
                    u = (_splitmix(seed, (b << 32) + 700 + j + 1) >> 11) / 9007199254740992.0
                    tok[b, j] = _sample(logits[b * q + j], float(np.float32(case["T"])),
                                        float(np.float32(case["p"])), case["k"], u)
        acc = torch.zeros(batch, dtype=torch.int32)
        for b in range(batch):
            for j in range(1, q):
                if int(drafts[b, j - 1]) != int(tok[b, j - 1]):
                    break
                acc[b] = j
        return tok, acc
    if kind == "attention":
        heads, dh = case["heads"], case["head_dim"]
        lens = _lens(case)
        k, v = next(_cache_kv(case, 1, heads, dh, True, g))
        qh = torch.randn((batch * q, heads * dh), generator=g, device="cuda").double().view(batch, q, heads, dh)
        out = torch.empty((batch, q, heads, dh), dtype=torch.float64, device="cuda")
        # the block's own slots hold what the cache held there: cached rows past a shorter sequence, else zeros
        for b, n in enumerate(lens):
            pad = max(0, n + q - k.shape[1])
            k1, v1 = (torch.cat([t[b, :n + q].double(), torch.zeros((pad, heads, dh), dtype=torch.float64,
                                                                    device="cuda")]) for t in (k, v))
            see = torch.ones((q, n + q), dtype=torch.bool, device="cuda").tril(n)
            out[b] = _attend(qh[b], k1, v1, see)
        return out.view(batch * q, heads * dh)
    sh = _model(case)
    w = _weights(case, g)
    if kind == "block":
        lens = _lens(case)
        caches = [[(k[b, :n].double(), v[b, :n].double()) for b, n in enumerate(lens)]
                  for k, v in _cache_kv(case, sh.n_layers, sh.n_heads, sh.head_dim, sh.dtype == "bf16", g)]
        depth, mask = _tree(q, case["tree"]) if case["tree"] else (None, None)
        return _forward(sh, w, caches, _tokens(sh, (batch, q), g), mask, depth, True)
    none = torch.zeros((0, sh.n_heads, sh.head_dim), dtype=torch.float64, device="cuda")
    caches = [[(none, none)] * batch for _ in range(sh.n_layers)]
    _forward(sh, w, caches, _tokens(sh, (batch, case["rows"]), g), None, None, False)
    return _forward(sh, w, caches, _tokens(sh, (batch, q), g), None, None, True)
