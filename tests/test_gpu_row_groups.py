"""Passes of three to eight row tiles, whose products the narrow kernel spreads over groups of as many workgroups: as
many groups as the device holds at once, whole rounds of the chiplets, and more tiles than groups.  The caches are those
of the wide kernel, whose shapes change over the same rows, bit for bit."""
import pytest

from paper_2605_13319_amd import inputs as I

pytestmark = pytest.mark.gpu

# four waves per workgroup (two workgroups per compute unit), eight, and phases with five
SHAPES = [I.ModelShape("groups-2048", 2, 2048, 16, 4, 128, 4096, 300), I.ModelShape("groups-4096", 2, 4096, 32, 8, 128, 4096, 300),
          I.ModelShape("groups-5120", 2, 5120, 40, 40, 128, 2560, 300)]

ROWS = (33, 64, 79, 96, 97, 112, 113, 128)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_groups_of_three_to_eight_row_tiles(shape):
    from paper_2605_13319_amd import nav
    model = nav.Model(shape, I.make_weights(shape, 71))
    for rows in ROWS:
        toks = I.make_tokens(rows + 1, shape.vocab, 72 + rows)
        pools = []
        for mode in (1, 2, 0):
            model.set_wide_gemm(mode)
            kv = nav.KVCache(model, max_seqs=1, n_blocks=rows // 16 + 2)
            kv.prefill(0, toks)
            pools.append(kv.pool.clone())
        assert bool((pools[0] == pools[1]).all()) and bool((pools[0] == pools[2]).all()), f"{rows} rows: the caches differ"


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_two_and_more_row_tiles_equal_passes_of_one(shape):
    """Two row tiles add their sums of squares in another kernel than one and three do (eight waves): the same bits."""
    from paper_2605_13319_amd import nav
    model = nav.Model(shape, I.make_weights(shape, 73))
    model.set_wide_gemm(1)
    toks = I.make_tokens(50, shape.vocab, 74)
    for rows in (17, 31, 32, 33, 48):
        kv, parts = (nav.KVCache(model, max_seqs=1, n_blocks=8) for _ in range(2))
        kv.prefill(0, toks[:rows + 1])
        for at in range(0, rows + 1, 16):
            parts.prefill(0, toks[at:min(at + 16, rows + 1)])
        assert bool((kv.pool == parts.pool).all()), f"{rows} rows: the caches differ"
