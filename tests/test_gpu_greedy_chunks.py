"""Greedy verification with rows cut into chunks over workgroups: vocabularies around the chunk edges (whole
and ragged vector loads, rows longer than all chunks at once), ties across chunks, rows of -inf and NaN, and
a second launch on the same context (the merge buffers are left zero)."""
import pytest
import torch

from paper_2403_18647_amd import binding as B
from paper_2403_18647_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [2, 1000, 8190, 8192, 8193, 8196, 16388, 131073, 140000])
@pytest.mark.parametrize("batch,q", [(1, 1), (3, 5), (1, 300)])
def test_chunks(vocab, batch, q):
    if vocab * batch * q > 2.5e7:
        pytest.skip("larger than the edges need")
    sh = synth.small_shape(n_layers=1, vocab=vocab)
    w = [torch.zeros(synth.tensor_shape(sh, n), device="cuda") for n in synth.tensor_names(sh)]
    ctx = B.Context(B.make_config(sh, batch, 512, q), w)
    g = torch.Generator(device="cuda")
    g.manual_seed(vocab + q)
    lg = torch.randn((batch * q, vocab), generator=g, device="cuda")
    n = -(-vocab // 8192)
    n = min(n, 16)
    chunk = (-(-vocab // n) + 3) // 4 * 4
    top = float(lg.max()) + 1
    for r in range(batch * q):   # the row's maximum twice or more, in different chunks where there are several
        ids = {(chunk - 1 + r) % vocab, (r * 37) % vocab, vocab - 1 - r % min(vocab, 3)}
        for i in ids:
            lg[r, i] = top
    if batch * q > 2:
        lg[1] = -float("inf")
        lg[2] = float("nan")
        lg[2, vocab // 2] = -5.0
    ref = torch.where(torch.isnan(lg), torch.full_like(lg, -float("inf")), lg).cpu()
    best = ref.max(-1).values[:, None]
    want = (ref == best).int().argmax(-1).int().view(batch, q)   # the first id that holds the maximum
    drafts = torch.randint(0, vocab, (batch, max(q - 1, 1)), generator=g, device="cuda", dtype=torch.int32)
    for b in range(batch):
        m = (q - 1) * b // max(1, batch - 1) if batch > 1 else q - 1
        drafts[b, :m] = want[b, :m].cuda()
        if m < q - 1:
            drafts[b, m] = (int(want[b, m]) + 1) % vocab
    tok = torch.empty((batch, q), dtype=torch.int32, device="cuda")
    acc = torch.empty(batch, dtype=torch.int32, device="cuda")
    for _ in range(2):
        tok.fill_(-1)
        acc.fill_(-1)
        B.sdsat_verify_greedy(ctx.handle, batch, q, lg, drafts if q > 1 else None, tok, acc)
        torch.cuda.synchronize()
        assert torch.equal(tok.cpu(), want)
        for b in range(batch):
            m = 0
            while q > 1 and m < q - 1 and int(drafts[b, m]) == int(want[b, m]):
                m += 1
            assert int(acc[b]) == m
    ctx.close()
