"""Attention of long prompts (four query tiles per workgroup, keys and values shared through LDS): against the checker by
the keys and values of the second layer, which follow from the first layer's attention, and by the logits of a row
behind them; and bit for bit against the streaming kernel, which takes the same blocks when they come alone.  Prompts end
at, before and behind the edges of tiles, steps, blocks and spans, for both head sizes and for head groups of one and of
several heads.  (Which kernel takes which pass, and with how many spans and workgroups: tests/test_attn_plan.py, on these cases.)"""
import numpy as np
import pytest

from oracle.nav import OracleSeq
from oracle.transformer import OracleModel
from paper_2605_13319_amd import inputs as I

# a block of 128 rows has 256 groups of four query tiles: enough for the prompt kernel by itself
BIG = [I.ModelShape("wide-64", 2, 512, 128, 16, 64, 512, 300), I.ModelShape("wide-128", 2, 512, 128, 16, 128, 512, 300)]
# a block by itself has 32 or 48 groups, which the streaming kernel takes
SMALL = [I.ModelShape("blocks-64", 2, 512, 16, 8, 64, 512, 300), I.ModelShape("blocks-128", 2, 1024, 24, 8, 128, 512, 300),
         I.ModelShape("blocks-mha", 2, 512, 16, 16, 128, 512, 300)]
# two layers at least: nothing reads the attention of a prompt's last layer
SHAPES = [I.ModelShape("attn-64", 2, 512, 16, 8, 64, 512, 300), I.ModelShape("attn-128", 2, 1024, 24, 8, 128, 512, 300)]
# prompt rows = tokens - 1: a full block; and one, 32, 33, 87 and 127 rows in a second
SHORT = [129, 130, 161, 162, 216, 256]
# (cached tokens, tokens of the call): a ragged third block; partials of a block's own workgroup and of several; spans of 256
# and more tokens, ten and more of them; workgroups that walk more than 64 steps
LONG = [(0, 400), (0, 700), (0, 2048), (0, 2049), (1, 513), (300, 450), (700, 1100), (700, 2020), (3000, 1050), (5000, 2048)]
STD = 0.05  # of the matrices: attention that matters
ROW_BOUND = 2.0 ** -8


def second_layer(shape, keys, values, rows):
    return np.concatenate([np.stack([np.asarray(a[r], np.float64).reshape(-1) for r in rows]) for a in (keys, values)], axis=1)


def row_errors(got, want):
    """Relative 2-norm per row.  Both sides round to bf16 numbers that agree but for the activations' 16 bits, so an
    element differs by one step (2^-7 of itself at most) or not at all, and few do: all differing by a step would be 2^-7
    at most, ROW_BOUND a quarter of them."""
    return np.linalg.norm(got - want, axis=1) / np.linalg.norm(want, axis=1)


def checker_rows(shape, weights, tokens):
    oseq = OracleSeq(OracleModel(shape, weights), tokens + 16)
    oseq.prefill(I.make_tokens(tokens, shape.vocab, 42 + tokens))
    return second_layer(shape, oseq.K[1], oseq.V[1], range(tokens - 1))


# (The prompt kernel takes the longest ones, and 300 tokens at head size 128; the streaming kernel the others, of fewer groups
# of tiles.)  The bound is the repository's for logits of bf16 models (the cache's rounding alone moves logits by 1e-3).
@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
@pytest.mark.parametrize("tokens", [129, 130, 161, 162, 216, 256, 300, 2049, 2060])
def test_prompt_attention_against_the_checker(shape, tokens):
    from paper_2605_13319_amd import nav
    w = I.make_weights(shape, 41)
    toks = I.make_tokens(tokens, shape.vocab, 42 + tokens)
    extra = I.make_tokens(2, shape.vocab, 43)
    oseq = OracleSeq(OracleModel(shape, w), tokens + 16)
    oseq.prefill(toks)
    want = oseq.forward_logits(extra)
    model = nav.Model(shape, w)
    kv = nav.KVCache(model, max_seqs=1, n_blocks=tokens // 16 + 2)
    kv.prefill(0, toks)
    got = kv.forward_logits(0, extra)
    print(shape.name, tokens, float(np.abs(got - want).max()), flush=True)
    assert np.abs(got - want).max() < 2e-2


@pytest.mark.gpu
@pytest.mark.parametrize("shape", BIG, ids=lambda s: s.name)
@pytest.mark.parametrize("tokens", SHORT + [300])
def test_second_layer_behind_prompt_attention_against_the_checker(shape, tokens):
    from paper_2605_13319_amd import nav
    w = I.make_weights(shape, 41, std=STD)
    model = nav.Model(shape, w)
    kv = nav.KVCache(model, max_seqs=1, n_blocks=tokens // 16 + 2)
    kv.prefill(0, I.make_tokens(tokens, shape.vocab, 42 + tokens))
    kvs = [kv.read_kv(0, 1, r) for r in range(tokens - 1)]
    got = second_layer(shape, [k for k, _ in kvs], [v for _, v in kvs], range(tokens - 1))
    err = row_errors(got, checker_rows(shape, w, tokens))
    print(shape.name, tokens, "largest error of a row", float(err.max()), flush=True)
    assert err.max() < ROW_BOUND


def _mistaken_softmax(kind):
    """The checker's softmax with a mistake planted: what a kernel that drops or adds tokens would return."""
    from oracle import transformer
    good = transformer.softmax_rows

    def bad(sc):
        sc = np.array(sc)
        m, n = sc.shape
        if kind == "zero":
            return np.zeros_like(sc)
        if kind == "own token":  # (the last rows' own key; the first token has no other)
            for r in range(max(0, 1 - (n - m)), m):
                sc[r, n - m + r] = -np.inf
        if kind == "first 32" and n > 64:
            sc[max(0, 33 - (n - m)):, :32] = -np.inf
        if kind == "token 100" and n > 101:
            sc[max(0, 101 - (n - m)):, 100] = -np.inf
        return good(sc)

    return bad


@pytest.mark.parametrize("shape", BIG, ids=lambda s: s.name)
@pytest.mark.parametrize("kind", ["zero", "own token", "first 32", "token 100"])
def test_mistakes_in_prompt_attention_exceed_the_bound(shape, kind, monkeypatch):
    w = I.make_weights(shape, 41, std=STD)
    want = checker_rows(shape, w, 162)
    monkeypatch.setattr("oracle.transformer.softmax_rows", _mistaken_softmax(kind))
    err = row_errors(checker_rows(shape, w, 162), want)
    assert err.max() > 4 * ROW_BOUND


def caches(shape, cached, calls):
    """The pool behind `cached` tokens (if any) and the calls of so many tokens each, one sequence per list of calls."""
    from paper_2605_13319_amd import nav
    model = nav.Model(shape, I.make_weights(shape, 41, std=STD))
    total = cached + sum(calls[0])
    text = I.make_tokens(total, shape.vocab, 43 + total)
    pools = []
    for sizes in calls:
        kv = nav.KVCache(model, max_seqs=1, n_blocks=total // 16 + 2)
        at = 0
        for n in ([cached] if cached else []) + sizes:
            kv.prefill(0, text[at:at + n])
            at += n
        pools.append(kv.pool.clone())
    return pools


def in_blocks(cached, tokens, rows):
    """Calls of `rows` rows each (a first call into an empty sequence has a row less than tokens)."""
    first = min(tokens, rows + (0 if cached else 1))
    sizes = [first]
    while sum(sizes) < tokens:
        sizes.append(min(rows, tokens - sum(sizes)))
    return sizes


@pytest.mark.gpu
@pytest.mark.parametrize("shape", BIG, ids=lambda s: s.name)
@pytest.mark.parametrize("tokens", SHORT + [257])
def test_prompt_equals_calls_of_32_rows(shape, tokens):
    """Up to 256 tokens of context are one span however few the rows, so every row has the bits that the streaming
    kernel gives it among 32."""
    a, b = caches(shape, 0, [[tokens], in_blocks(0, tokens, 32)])
    assert bool((a == b).all())


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SMALL, ids=lambda s: s.name)
@pytest.mark.parametrize("cached,tokens", LONG)
def test_prompt_equals_its_blocks_alone(shape, cached, tokens):
    a, b = caches(shape, cached, [[tokens], in_blocks(cached, tokens, 128)])
    assert bool((a == b).all())
