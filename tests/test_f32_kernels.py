"""The fp32 model's kernels at the sizes where their tiles, splits and row blocks end, against the checker."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2605_13319_amd import inputs as I
from tests import isa_lint
from tests.helpers import oracle_side

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def test_no_early_read_of_matrix_core_results_across_blocks(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = tmp_path / "f32.s"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-S", "--cuda-device-only", "-o", str(out),
                    os.path.join(ROOT, "paper_2605_13319_amd", "csrc", "kernels_f32.hip")], check=True, capture_output=True)
    assert "v_mfma_f32_16x16x4" in out.read_text()
    assert isa_lint.check_mfma(str(out)) == 0


# (layers, d_model, query heads, KV heads, head_dim, d_ffn, vocab): head sizes with and without the
# matrix-core attention (multiples of 16 or not), widths that are no multiple of the 16-column blocks,
# rows of W_o that do not start on 16-byte boundaries (2 and 6 columns), ragged last tiles everywhere
SHAPES = [(2, 36, 3, 1, 20, 44, 99), (2, 52, 6, 2, 48, 20, 130), (1, 8, 1, 1, 2, 4, 3), (1, 64, 2, 2, 128, 64, 257),
          (2, 132, 3, 3, 2, 60, 65), (1, 260, 8, 2, 16, 140, 1025)]


@pytest.mark.gpu
@pytest.mark.parametrize("dims", SHAPES)
@pytest.mark.parametrize("prompt,ks", [(2, (1, 31)), (130, (15, 16)), (257, (4, 17))])
def test_odd_shapes_against_the_checker(dims, prompt, ks):
    """Prompts of one row, of one block and a row, and of two blocks and a second split of the
    context, the last token pending; then rounds of 2, 32, 16, 17, 5 and 18 rows."""
    from paper_2605_13319_amd import nav
    shape = I.ModelShape("f32-odd", *dims, dtype=I.DTYPE_F32)
    w = I.make_weights(shape, 31, std=0.08)
    toks = I.make_tokens(prompt, shape.vocab, 32)
    oseq = oracle_side(shape, w, toks, prompt + 80)
    model = nav.Model(shape, w)
    kv = nav.KVCache(model, max_seqs=1, n_blocks=(prompt + 80) // 16 + 1)
    kv.prefill(0, toks)
    print(dims, prompt, "prompt cached", flush=True)
    for layer in range(shape.n_layers):
        for pos in sorted({0, (prompt - 2) // 2, prompt - 2}):
            k_gpu, v_gpu = kv.read_kv(0, layer, pos)
            np.testing.assert_allclose(k_gpu, oseq.K[layer][pos].reshape(-1), rtol=0, atol=1e-5)
            np.testing.assert_allclose(v_gpu, oseq.V[layer][pos].reshape(-1), rtol=0, atol=1e-5)
    for k in ks:
        d = I.make_tokens(k, shape.vocab, 33 + k)
        z, z_ref = kv.forward_logits(0, d), oseq.forward_logits(d)
        assert float(np.abs(z - z_ref).max()) <= 1e-4
        # token matching on a text whose first draft is the target's own choice where that is clear
        top = np.sort(z_ref[0])[-2:] if shape.vocab > 1 else np.array([0.0, 1.0])
        if top[1] - top[0] > 1e-3:
            d0 = int(z_ref[0].argmax())
            z2 = oseq.forward_logits([d0])[1]
            top2 = np.sort(z2)[-2:]
            if top2[1] - top2[0] > 1e-3:
                a, nxt = kv.nav_verify(0, [d0, (int(z2.argmax()) + 1) % shape.vocab])
                assert (a, nxt) == (1, int(z2.argmax()))
                kv.rollback(0, prompt)


@pytest.mark.gpu
def test_rows_of_a_block_equal_rows_of_shorter_blocks():
    """A row's results do not depend on how many rows share its launch (1, 2 row tiles, 4 workgroups of
    rows): the same prompt in one call and token by token leaves the same cache, bit for bit."""
    from paper_2605_13319_amd import nav
    shape = I.ModelShape("f32-blocks", 2, 64, 4, 2, 32, 72, 50, dtype=I.DTYPE_F32)
    model = nav.Model(shape, I.make_weights(shape, 41, std=0.08))
    kv = nav.KVCache(model, max_seqs=2, n_blocks=2 * 12)
    toks = I.make_tokens(150, shape.vocab, 42)
    kv.prefill(0, toks)
    for i in (0, 1, 20, 60, 117):  # 1, 19, 40, 57 and 33 rows at a time
        j = {0: 1, 1: 20, 20: 60, 60: 117, 117: 150}[i]
        kv.prefill(1, toks[i:j])
    for layer in range(2):
        for pos in range(0, 149, 4):
            for a, b in zip(kv.read_kv(0, layer, pos), kv.read_kv(1, layer, pos)):
                np.testing.assert_array_equal(a, b)
