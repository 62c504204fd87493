"""Prompt ingestion in passes of up to 2048 rows against passes of 128 rows on the narrow GEMM kernel:
the same cache, bit for bit, whatever tiles, splits of K and row blocks the wide kernel takes."""
import pytest

from paper_2605_13319_amd import inputs as I

pytestmark = pytest.mark.gpu

# K of the products: 512 (one slice), 1536 (W = 3), 4608 (W = 3, three phases), 7168 (W = 7, two phases),
# 2048 and 4096 (W = 4, 8), 14336 (W = 7, four phases); 512 .. 28672 weight rows
SHAPES = [I.ModelShape("prompt-512", 2, 512, 8, 2, 64, 1536, 300), I.ModelShape("prompt-mha", 2, 512, 4, 4, 128, 4608, 300),
          I.ModelShape("prompt-2048", 2, 2048, 16, 4, 128, 7168, 300), I.ModelShape("prompt-4096", 2, 4096, 32, 8, 128, 14336, 300)]


# rows of the first pass (tokens - 1): three and four row tiles (by product narrow or wide), five, a full and a ragged last row
# block, one row in the last 16, and (2049 and more tokens) a second pass of one row and of a few hundred
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_long_passes_equal_short_ones(shape):
    from paper_2605_13319_amd import nav
    model = nav.Model(shape, I.make_weights(shape, 61))
    for tokens in (34, 50, 65, 66, 97, 129, 130, 146, 258, 334, 690, 2049, 2050, 2381):
        toks = I.make_tokens(tokens, shape.vocab, 62 + tokens)
        pools = []
        for mode in (1, 0, 2):
            model.set_wide_gemm(mode)
            kv = nav.KVCache(model, max_seqs=1, n_blocks=(tokens + 15) // 16 + 1)
            kv.prefill(0, toks)
            pools.append(kv.pool.clone())
        print(shape.name, tokens, flush=True)
        assert bool((pools[0] == pools[1]).all()) and bool((pools[0] == pools[2]).all()), f"{tokens} tokens: the caches differ"


def test_a_turn_behind_a_cached_context_equals_one_prompt():
    """A prompt in one call and in calls of 1000, 37, 333 and 131 tokens (each call's first row is the
    pending token of the call before): the products see other row blocks, the attention other splits of
    the context, so the caches agree to a bf16 step."""
    import torch
    from paper_2605_13319_amd import nav
    shape = SHAPES[0]
    model = nav.Model(shape, I.make_weights(shape, 61))
    toks = I.make_tokens(1501, shape.vocab, 70)
    kv = nav.KVCache(model, max_seqs=2, n_blocks=2 * 95)
    kv.prefill(0, toks)
    for i, j in ((0, 1000), (1000, 1037), (1037, 1370), (1370, 1501)):
        kv.prefill(1, toks[i:j])
    # (blocks are handed out in order: the second sequence's follow the first's)
    p = kv.pool.view(torch.bfloat16).view(shape.n_layers, 2, 2 * 95, -1).float()
    full = 1500 // 16
    a, b = p[:, :, :full], p[:, :, full + 1:2 * full + 1]
    assert float((a - b).abs().max()) <= 2.0 ** -7 * float(a.abs().max())
    assert float((a != b).float().mean()) < 0.02
