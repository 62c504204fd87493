"""Every form of the wide products' kernel that passes of the 1B, 8B and 13B widths and of two others take, against the narrow kernel: the
same caches, bit for bit, and (the LM head, which only calls of several clients run on it) the same probabilities.
tests/test_gemm_plan.py counts the forms."""
import numpy as np
import pytest

from paper_2605_13319_amd import inputs as I
from tests.test_gpu_prompt import SHAPES

pytestmark = pytest.mark.gpu

# rows of a prompt's first pass: what tests/test_gpu_prompt.py and tests/test_gpu_row_groups.py leave out
ROWS = [(SHAPES[2], (513, 577, 673, 1281)), (SHAPES[3], (193, 769, 897, 1089, 1153, 1281, 1537, 1601)),
        (I.ModelShape("prompt-5120", 2, 5120, 40, 40, 128, 13824, 300), (33, 65, 129, 257, 321, 577, 769, 897, 1217, 1537)),
        (I.ModelShape("prompt-3072", 2, 3072, 24, 8, 128, 8192, 300), (129, 193, 289, 673, 801, 1281, 1345, 1537)),
        (I.ModelShape("prompt-6144", 2, 6144, 48, 8, 128, 1024, 300), (33, 65, 97, 129, 321))]


@pytest.mark.parametrize("shape,rows", ROWS, ids=[s.name for s, _ in ROWS])
def test_caches_of_the_wide_kernel_are_the_narrow_ones(shape, rows):
    from paper_2605_13319_amd import nav
    model = nav.Model(shape, I.make_weights(shape, 61))
    for n in rows:
        toks = I.make_tokens(n + 1, shape.vocab, 162 + n)
        pools = []
        for mode in (1, 0, 2):
            model.set_wide_gemm(mode)
            kv = nav.KVCache(model, max_seqs=1, n_blocks=n // 16 + 2)
            kv.prefill(0, toks)
            pools.append(kv.pool.clone())
        print(shape.name, n, flush=True)
        assert bool((pools[0] == pools[1]).all()) and bool((pools[0] == pools[2]).all()), f"{n} rows: the caches differ"


HEADS = [I.ModelShape("head-2048", 1, 2048, 32, 8, 64, 512, 32000), I.ModelShape("head-5120", 1, 5120, 40, 40, 128, 512, 32000)]
HEAD_ROWS = (33, 64, 112, 144, 176, 192, 256)


@pytest.mark.parametrize("shape", HEADS, ids=lambda s: s.name)
def test_heads_of_several_clients_leave_the_probabilities_of_one(shape):
    """The draft distribution gives every draft a ratio p/q of 1/2 to 1e-4 by the probabilities p of a pass of its own, and the
    uniforms are 1/2: just above it all drafts pass, just below it at one position that draft does not.  (p in 64 bits from
    32-bit logits: 1e-6 off the kernel's; a wrong column or row of the product is far more.)"""
    from paper_2605_13319_amd import nav
    model = nav.Model(shape, I.make_weights(shape, 64))
    kv = nav.KVCache(model, max_seqs=16, n_blocks=16 * 5)
    lens = [17 + 2 * s for s in range(16)]
    for s, n in enumerate(lens):
        kv.prefill(s, I.make_tokens(n, shape.vocab, 65 + s))
    for rows in HEAD_ROWS:
        n = max(2, rows // 16)
        per = [rows // n + (s < rows % n) for s in range(n)]  # rows of the clients
        drafts, probs = [], []
        for s in range(n):
            d = [int(t) for t in np.random.default_rng(1000 * rows + s).integers(0, shape.vocab, per[s] - 1)]
            z = np.asarray(kv.forward_logits(s, d), dtype=np.float64)
            p = np.exp(z - z.max(axis=1, keepdims=True))
            drafts.append(d)
            probs.append((p / p.sum(axis=1, keepdims=True))[np.arange(len(d)), d])
        for fails in (False, True):
            qs, want = [], []
            for s, (d, p) in enumerate(zip(drafts, probs)):
                at = (3 * s + rows) % len(d) if fails else len(d)
                ratio = np.where(np.arange(len(d)) == at, 0.5 * (1 - 1e-4), 0.5 * (1 + 1e-4))
                q = np.full((len(d), shape.vocab), 1e-9, dtype=np.float32)
                q[np.arange(len(d)), d] = p / ratio
                qs.append(q)
                want.append(at)
            a, _ = kv.nav_verify_batch(list(range(n)), drafts, qs, [[0.5] * (len(d) + 1) for d in drafts])
            for s in range(n):
                kv.rollback(s, lens[s])
            assert list(a) == want, f"{rows} rows, one draft fails: {fails}"
        print(shape.name, rows, flush=True)
