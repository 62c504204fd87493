"""Down projections whose waves take several K slices and a single tile: the next slice's weights and
activations are requested while the current one is multiplied."""
import numpy as np
import pytest

from paper_2605_13319_amd import inputs as I
from tests.helpers import oracle_side

pytestmark = pytest.mark.gpu


# slices of 512 columns (waves x slices per wave): 9 = 3 x 3, 10 = 5 x 2, 11 = 1 x 11, 14 = 7 x 2, 32 = 8 x 4;
# one tile and two tiles of rows, the last row of a tile and the first of the next, and a single row
@pytest.mark.parametrize("slices", [9, 10, 11, 14, 32])
def test_down_projection_of_several_slices(slices):
    from paper_2605_13319_amd import nav
    shape = I.ModelShape(f"down-{slices}", 2, 512, 8, 2, 64, 512 * slices, 300)
    w = I.make_weights(shape, 81)
    toks = I.make_tokens(37, shape.vocab, 82)
    oseq = oracle_side(shape, w, toks, 37 + 64)
    model = nav.Model(shape, w)
    kv = nav.KVCache(model, max_seqs=1, n_blocks=8)
    kv.prefill(0, toks)
    first = None
    for rows in (32, 17, 16, 9, 5, 1):
        d = I.make_tokens(32, shape.vocab, 83)[:rows - 1]
        z = kv.forward_logits(0, d)
        err = float(np.abs(z - oseq.forward_logits(d)).max())
        print(f"{slices} slices, {rows} rows: err {err:.2e}", flush=True)
        assert err <= 2e-2  # the bound of a bf16 model's logits against the checker with a bf16 cache
        # the order of a row's additions does not depend on how many rows the pass has
        first = z if first is None else first
        assert np.array_equal(z, first[:rows])
