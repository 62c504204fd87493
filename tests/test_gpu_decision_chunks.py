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
