"""The decision step where its chunks and its sweeps end, bit-exact with the checker."""
import numpy as np
import pytest

from oracle.spec_sampling import spec_accept as oracle_accept
from paper_2605_13319_amd import inputs as I


@pytest.mark.gpu
@pytest.mark.parametrize("vocab", [1, 2, 63, 64, 65, 2049, 131072, 131073, 131137])
@pytest.mark.parametrize("k", [1, 3])
def test_decision_at_the_ends_of_its_chunks(vocab, k):
    """Vocabularies around the 64 chunks and around what a workgroup sweeps at once (2048 tokens per
    chunk); uniforms at both ends so that the first and the last token are drawn."""
    import torch
    from paper_2605_13319_amd import nav
    p = I.make_random_probs(k + 1, vocab, 50 + vocab)
    q = I.make_random_probs(k, vocab, 51 + vocab)
    d = I.make_tokens(k, vocab, 52)
    pd, qd = torch.from_numpy(p).cuda(), torch.from_numpy(q).cuda()
    for last in (0.0, 0.5, 1 - 2.0 ** -24):
        for first in (0.0, 1 - 2.0 ** -24):
            u = np.array([0.0] * (k - 1) + [first, last], dtype=np.float32)
            assert nav.spec_accept(pd, qd, d, u) == oracle_accept(p, q, d, u)


@pytest.mark.gpu
@pytest.mark.parametrize("first", [0, 8, 13])
def test_draw_takes_the_smallest_token_above_the_threshold(first):
    """The drawn token is the smallest whose running 64-bit sum exceeds the threshold, also where the
    sum comes back below it further on (four weights of 2^62 add up to 0): all inside the first of the
    64 chunks (16 tokens), in one thread's eight tokens, in the second thread's, and across two threads
    and the chunk's end.  Twice in a row: the first call leaves its scratch as it found it."""
    import torch
    from paper_2605_13319_amd import nav
    vocab, k = 1024, 1
    p = np.zeros((k + 1, vocab), dtype=np.float32)
    p[0, 5] = 0.5
    p[1, 0] = 0.25 if first else 0.0
    p[1, first:min(first + 4, 16)] = 2.0 ** 22
    if first < 13:
        p[1, first + 4] = 1.0
    else:
        p[1, 900] = 2.0 ** 22 + 0.5
    q = np.full((k, vocab), 1.0 / vocab, dtype=np.float32)
    u = np.array([0.0, 0.5], dtype=np.float32)
    w = [int(float(x) * 2.0 ** 40) for x in p[1]]
    T = ((sum(w) % 2 ** 64) * 2 ** 23) >> 24
    run, want = 0, None
    for j, x in enumerate(w):
        run = (run + x) % 2 ** 64
        if want is None and run > T:
            want = j
    assert want == first
    pd, qd = torch.from_numpy(p).cuda(), torch.from_numpy(q).cuda()
    result = torch.zeros(2, dtype=torch.int32, device="cuda")
    for _ in range(2):
        assert nav.spec_accept(pd, qd, [5], u) == (1, want)
        nav.spec_accept_static(pd, qd, [5], u, result)
        assert result.tolist() == [1, want]


@pytest.mark.gpu
@pytest.mark.parametrize("vocab", [3, 65, 2049, 131072, 131073, 200001])
def test_decision_from_logits_at_the_ends_of_its_sweeps(vocab):
    """A sampled round on the logits of a model: vocabularies below the 64 chunks, and on both sides of
    131072, up to which the softmax statistics hold a chunk in registers.  The tests sit 1e-3 on either
    side of p/q = 1/2, and the drawn token's interval of the distribution function must meet the
    uniform to 1e-4: fp32 sums over a vocabulary are about 1e-6 off, a missed chunk would be 1e-2."""
    import torch
    from paper_2605_13319_amd import nav
    shape = I.ModelShape(f"vocab-{vocab}", 1, 64, 2, 1, 16, 64, vocab, dtype=I.DTYPE_F32)
    w = I.make_weights(shape, 91, std=0.1)
    toks = I.make_tokens(9, vocab, 92)
    model = nav.Model(shape, w)
    kv = nav.KVCache(model, max_seqs=1, n_blocks=2)
    kv.prefill(0, toks)
    drafts = I.make_tokens(2, vocab, 93)
    z = kv.forward_logits(0, drafts).astype(np.float64)
    p = np.exp(z - z.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    for i in range(2):  # drafts with p < 1/2, so that there is a q of twice the size
        if p[i, drafts[i]] > 0.45:
            drafts[i] = int(p[i].argmin())
    z = kv.forward_logits(0, drafts).astype(np.float64)
    p = np.exp(z - z.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    q = 0.5 * p[:2]
    for i in range(2):  # twice p at the draft, half of it elsewhere, the rest of the mass on one more token
        q[i, drafts[i]] = 2.0 * p[i, drafts[i]]
        other = (drafts[i] + 1) % vocab
        q[i, other] += 1.0 - q[i].sum()
    q = q.astype(np.float32)
    qd = torch.from_numpy(q).cuda()
    for draw in (2.0 ** -24, 0.3, 0.77, 1 - 2.0 ** -24):
        for tests, want in (((0.4995, 0.5005), 1), ((0.4995, 0.4995), 2), ((0.5005, 0.0), 0)):
            a, nxt = kv.nav_verify(0, drafts, qd, np.array([*tests, draw], dtype=np.float32))
            kv.rollback(0, len(toks))
            assert a == want
            law = p[2] if a == 2 else np.maximum(0.0, p[a] - q[a].astype(np.float64))
            cdf = np.cumsum(law) / law.sum()
            lo = cdf[nxt - 1] if nxt > 0 else 0.0
            assert lo - 1e-4 <= draw <= cdf[nxt] + 1e-4, (tests, draw, nxt, lo, cdf[nxt])
            assert law[nxt] > 0
