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
TOKENS = (34, 50, 65, 66, 97, 129, 130, 146, 258, 334, 690, 2049, 2050, 2381)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_long_passes_equal_short_ones(shape):
    from paper_2605_13319_amd import nav
    model = nav.Model(shape, I.make_weights(shape, 61))
    for tokens in TOKENS:
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


# tokens cached first (behind them a block of 128 rows takes 8 or 16 splits of the context), and tokens of
# the call itself: a full block and a row, a ragged last block of a few rows (cut finer than the others),
# a longer ragged one, and a second pass of one row
TOKENS_BEHIND = (129, 270, 700, 2049)  # (as many rows: the pending token and all but the last)


@pytest.mark.parametrize("shape", SHAPES[:3], ids=lambda s: s.name)
@pytest.mark.parametrize("cached", [4500, 9001])
def test_long_passes_behind_a_cached_context_equal_short_ones(shape, cached):
    from paper_2605_13319_amd import nav
    model = nav.Model(shape, I.make_weights(shape, 61))
    first = I.make_tokens(cached, shape.vocab, 71)
    for tokens in TOKENS_BEHIND:
        toks = I.make_tokens(tokens, shape.vocab, 72 + tokens)
        pools = []
        for mode in (1, 0, 2):
            model.set_wide_gemm(mode)
            kv = nav.KVCache(model, max_seqs=1, n_blocks=(cached + tokens + 15) // 16 + 1)
            kv.prefill(0, first)
            kv.prefill(0, toks)
            pools.append(kv.pool.clone())
        print(shape.name, cached, tokens, flush=True)
        assert bool((pools[0] == pools[1]).all()) and bool((pools[0] == pools[2]).all()), f"{tokens} tokens: the caches differ"


def test_context_beyond_the_streaming_attention():
    """Behind 131072 tokens prompts run in passes of 128 rows and every pass on the split kernels.  One
    layer, so that the keys and values of all tokens follow from their embeddings, and weights large
    enough for peaked attention (the logits without it are far off): logits of passes of 1, 16 and 17
    rows against 64 bits, the bound that of a bf16 model's logits."""
    import torch
    from paper_2605_13319_amd import nav
    shape = I.ModelShape("far", 1, 512, 8, 1, 64, 512, 300)
    w = I.make_weights(shape, 95, std=0.08)
    n = 131072 + 200
    toks = I.make_tokens(n, shape.vocab, 96)
    extra = I.make_tokens(16, shape.vocab, 97)
    model = nav.Model(shape, w)
    kv = nav.KVCache(model, max_seqs=1, n_blocks=(n + 16 + 15) // 16 + 1)
    kv.prefill(0, toks[:n - 150])
    kv.prefill(0, toks[n - 150:])

    def wide(a):
        t = torch.from_numpy(a.view("int16")).cuda().view(torch.bfloat16) if a.dtype.itemsize == 2 else torch.from_numpy(a).cuda()
        return t.double()

    h, g = shape.head_dim, shape.n_q_heads
    text = torch.tensor(list(toks) + list(extra), device="cuda")
    x = wide(w["tok_emb"])[text]
    theta = shape.rope_base ** (-2.0 * torch.arange(h // 2, dtype=torch.float64, device="cuda") / h)
    ang = torch.arange(len(text), device="cuda").double()[:, None] * theta
    cos, sin = torch.cos(ang), torch.sin(ang)

    def norm(v, gain):
        return v * torch.rsqrt(v.square().mean(-1, keepdim=True) + shape.rms_eps) * wide(gain)

    def rotate(v, c, s):
        a, b = v[..., : h // 2], v[..., h // 2:]
        return torch.cat([a * c - b * s, b * c + a * s], dim=-1)

    y = norm(x, w["attn_norm"][0])
    keys = rotate(y @ wide(w["wk"][0]).t().contiguous(), cos, sin).bfloat16().double()
    vals = (y @ wide(w["wv"][0]).t().contiguous()).bfloat16().double()
    rows = slice(n - 1, n + 16)
    q = rotate((y[rows] @ wide(w["wq"][0]).t().contiguous()).view(17, g, h), cos[rows][:, None], sin[rows][:, None])
    sc = (q.reshape(17 * g, h) @ keys.t().contiguous()).view(17, g, -1) / h ** 0.5
    later = torch.arange(n + 16, device="cuda")[None, :] > torch.arange(n - 1, n + 16, device="cuda")[:, None]
    p = torch.softmax(sc.masked_fill(later[:, None, :], float("-inf")), dim=-1)
    o = (p.view(17 * g, -1) @ vals).view(17, g * h)

    def logits(attended):
        z = x[rows] + attended @ wide(w["wo"][0]).t().contiguous()
        f = norm(z, w["ffn_norm"][0])
        f = torch.nn.functional.silu(f @ wide(w["w_gate"][0]).t().contiguous()) * (f @ wide(w["w_up"][0]).t().contiguous())
        z = z + f @ wide(w["w_down"][0]).t().contiguous()
        return (norm(z, w["final_norm"]) @ wide(w["lm_head"]).t().contiguous()).cpu().numpy()

    ref = logits(o)
    assert abs(ref - logits(0.0 * o)).max(axis=1).min() > 0.2
    got = {}
    for m in (1, 16, 17):
        got[m] = kv.forward_logits(0, extra[:m - 1])
        err = float(abs(got[m] - ref[:m]).max())
        print(f"{m} rows behind {n} tokens: err {err:.2e}", flush=True)
        assert err <= 2e-2
    assert (got[1] == got[17][:1]).all() and (got[16] == got[17][:16]).all()
