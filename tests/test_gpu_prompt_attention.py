"""Attention of prompt blocks (four query tiles per workgroup, keys and values shared through LDS) against the
checker: logits of a row behind prompts whose rows end at, before and behind the edges of tiles, steps, blocks and
spans, for both head sizes and for head groups of several rows per tile.  The bound is the repository's for
bf16 models (2e-2; the cache's rounding alone moves logits by 1e-3)."""
import numpy as np
import pytest

from oracle.nav import OracleSeq
from oracle.transformer import OracleModel
from paper_2605_13319_amd import inputs as I

pytestmark = pytest.mark.gpu

# 8 KV heads x 16 or 32 query tiles per full block: enough tiles for the prompt kernel
SHAPES = [I.ModelShape("attn-64", 2, 512, 16, 8, 64, 512, 300), I.ModelShape("attn-128", 1, 1024, 24, 8, 128, 512, 300)]


# prompt rows = tokens - 1: a full block; and one, 32 (another kernel, same launch), 33, 87 and 127 rows in a second; a ragged
# third; 64 steps exactly and a step more in one span, two spans of the last block
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
