"""Nucleus verification where only the ids that can be in the nucleus are gathered: vocabulary edges, flat and
peaked rows (nearly all ids left, a handful, one), ties at the threshold, -inf ids and temperatures that push
the candidate range to either path, against the oracle's sampler on the same uniforms."""
import numpy as np
import pytest
import torch

from oracle import sampling as S
from paper_2403_18647_amd import binding as B
from paper_2403_18647_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [3, 1000, 1025, 8193, 32016, 32768])
@pytest.mark.parametrize("temp,p", [(0.05, 0.95), (0.8, 0.95), (1.0, 0.9), (1.0, 0.5), (3.0, 0.99), (1e30, 0.5)])
def test_few(vocab, temp, p):
    q = 5
    sh = synth.small_shape(n_layers=1, vocab=vocab)
    w = [torch.zeros(synth.tensor_shape(sh, n), device="cuda") for n in synth.tensor_names(sh)]
    ctx = B.Context(B.make_config(sh, 1, 64, q), w)
    rng = np.random.default_rng(vocab)
    lg = rng.standard_normal((q, vocab)).astype(np.float32) * 4
    lg[1] = np.round(lg[1])                     # ties everywhere, at the threshold too
    lg[2, vocab // 3:] = -np.inf                # ids that cannot be drawn
    lg[3] = 0.25 * lg[3]                        # flat: thousands of candidates
    lg[4, vocab - 1] = 60.0                     # one id holds the mass
    d = torch.from_numpy(lg).cuda()
    pos0 = torch.tensor([17], dtype=torch.int32, device="cuda")
    drafts = torch.zeros((1, q - 1), dtype=torch.int32, device="cuda")
    tok = torch.empty((1, q), dtype=torch.int32, device="cuda")
    acc = torch.empty(1, dtype=torch.int32, device="cuda")
    for seed in range(6):
        B.sdsat_verify_nucleus(ctx.handle, 1, q, d, drafts, temp, p, 0, seed, pos0, tok, acc)
        torch.cuda.synchronize()
        got = tok.cpu().numpy()[0]
        for j in range(q):
            want, margin = S.sample(lg[j], float(np.float32(temp)), float(np.float32(p)), 0, S.uniform(seed, 0, 17 + j))
            # a draw this close to a decision boundary may go either way with float64 sums in another order
            assert int(got[j]) == int(want) or margin < 1e-9, (vocab, temp, p, seed, j)
    ctx.close()


# p; ids at each logit (the rest at -20) at T = 1, V = 32016.  First cut -9.0 (p 0.95) or -13.0 (p 0.99), second
# -14.4 or -16.0; 8192 ids fit; beyond 2048 above the first cut the float32 sum decides.
ROUTES = {
    "fits exactly": (0.95, {0.0: 1, -5.0: 8191, -9.2: 20000}),
    "one too many": (0.95, {0.0: 1, -5.0: 8192, -9.2: 20000}),
    "tail too heavy, second cut too many": (0.95, {0.0: 1, -5.0: 3000, -9.2: 29015}),
    "tail too heavy, seen after the sums": (0.95, {0.0: 1, -5.0: 1000, -9.2: 31015}),
    "second cut, few above the first": (0.95, {0.0: 1, -6.0: 20, -9.2: 5000}),
    "second cut, many above the first": (0.95, {0.0: 1, -8.5: 2100, -9.2: 6000}),
    "second cut fits exactly": (0.95, {0.0: 1, -6.0: 20, -9.2: 8171}),
    "p 0.99": (0.99, {0.0: 1, -8.0: 300, -12.9: 6000, -13.2: 20000}),
    "p 0.99, second cut": (0.99, {0.0: 1, -13.2: 8000}),
}


@pytest.mark.parametrize("name", list(ROUTES))
def test_routes(name):
    """Rows on either side of each decision of the gathered sampler (levels spread a little, so that few ids tie)."""
    p, levels = ROUTES[name]
    vocab, rng = 32016, np.random.default_rng(7)
    lg = np.full((4, vocab), -20.0, np.float32)
    for row in lg:
        ids, at = rng.permutation(vocab), 0
        for level, n in levels.items():
            row[ids[at:at + n]] = level + (0.05 * rng.random(n) if n > 1 else 0)
            at += n
    for seed in range(4):
        got = _verify(lg, 1.0, p, seed)
        for j in range(4):
            want, margin = S.sample(lg[j], 1.0, float(np.float32(p)), 0, S.uniform(seed, 0, 17 + j))
            assert got[j] == int(want) or margin < 1e-9, (name, seed, j)


def _verify(lg, temp, p, seed):
    q, vocab = lg.shape
    sh = synth.small_shape(n_layers=1, vocab=vocab)
    w = [torch.zeros(synth.tensor_shape(sh, n), device="cuda") for n in synth.tensor_names(sh)]
    ctx = B.Context(B.make_config(sh, 1, 64, q), w)
    pos0 = torch.tensor([17], dtype=torch.int32, device="cuda")
    drafts = torch.zeros((1, q - 1), dtype=torch.int32, device="cuda")
    tok = torch.empty((1, q), dtype=torch.int32, device="cuda")
    acc = torch.empty(1, dtype=torch.int32, device="cuda")
    B.sdsat_verify_nucleus(ctx.handle, 1, q, torch.from_numpy(lg).cuda(), drafts, temp, p, 0, seed, pos0, tok, acc)
    torch.cuda.synchronize()
    ctx.close()
    return tok.cpu().numpy()[0]


@pytest.mark.parametrize("vocab", [3, 1000, 8192, 8193, 32016, 32768])
@pytest.mark.parametrize("p", [0.5, 0.95])
def test_infinite_temperature(vocab, p):
    """Every weight is 1: the nucleus is the p V largest logits (ties at the threshold kept), drawn uniformly."""
    rng = np.random.default_rng(vocab)
    lg = rng.standard_normal((4, vocab)).astype(np.float32) * 4
    lg[1] = np.round(lg[1])
    got = _verify(lg, float("inf"), p, 5)
    for j in range(4):
        srt = np.sort(lg[j])[::-1]
        n = int(np.ceil(float(np.float32(p)) * vocab))   # whole sums: the threshold is exact
        ids = np.nonzero(lg[j] >= srt[n - 1])[0]
        assert got[j] == ids[int(S.uniform(5, 0, 17 + j) * len(ids))], (vocab, p, j)


@pytest.mark.parametrize("vocab", [3, 1000, 8192, 8193, 32016, 32768])
def test_no_finite_mass(vocab):
    """Rows whose mass is no number have no threshold: the last id, never one outside the vocabulary."""
    rng = np.random.default_rng(vocab)
    lg = rng.standard_normal((6, vocab)).astype(np.float32) * 4
    lg[0, 0] = np.nan
    lg[1, vocab // 2] = -np.float32(np.nan)
    lg[2, vocab - 1] = np.inf
    lg[3] = -np.inf
    lg[4] = np.nan
    lg[5, 1] = np.inf
    lg[5, 2] = np.inf
    for temp, p in ((0.8, 0.95), (float("inf"), 0.5)):
        got = _verify(lg, temp, p, 3)
        if temp < np.inf:
            assert (got == vocab - 1).all(), got
        assert ((got >= 0) & (got < vocab)).all(), got
