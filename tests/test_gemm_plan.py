"""Which forms of the wide products' kernel the passes of a model take (CPU), and that the GPU tests which compare that
kernel's results with the narrow one's reach all of them, so that a change of the time models cannot leave one untested."""
import os
import shutil
import subprocess

import pytest

from paper_2605_13319_amd import inputs as I

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_13319_amd", "csrc")

PLANS = r"""
#include <stdio.h>
#include <stdlib.h>
#include "attn_plan.h"
#include "gemm_plan.h"
using namespace pipesd;
// d_model q_dim kv_dim d_ffn vocab, then (rows, mode) pairs: per pair and product on the wide kernel: rows, product, n-tiles
// per workgroup, row tiles per wave, whole, phases, bit set of the row tiles that a wave has
int main(int argc, char** argv) {
  const int d = atoi(argv[1]), qd = atoi(argv[2]), kvd = atoi(argv[3]), F = atoi(argv[4]), V = atoi(argv[5]), n_cu = 256;
  const int nk[5][2] = {{qd + 2 * kvd, d}, {d, qd}, {2 * F, d}, {d, F}, {V, d}};
  size_t ws = 0;
  for (int i = 0; i < 5; ++i) ws = std::max(ws, gemm_wide_workspace_bytes(nk[i][0], nk[i][1], i < 4 ? kMaxPromptRows : kMaxPassRows));
  for (int a = 6; a + 1 < argc; a += 2) {
    const int rows = atoi(argv[a]), rt = (rows + 15) / 16;
    for (int i = 0; i < (rows <= kMaxPassRows ? 5 : 4); ++i) {
      const int N = nk[i][0], K = nk[i][1];
      const GemmPlan p = gemm_narrow_plan(N, K, rt, n_cu);
      if (!gemm_takes_wide(p, rt, i != 1 && i != 3, atoi(argv[a + 1]), n_cu, ws)) continue;
      const WidePlan w = wide_plan(N, K, rt, n_cu, ws);
      if (w.ct == 0) return 1;
      unsigned tiles = 0;
      for (int rb = 0; rb < w.nrb; ++rb)
        for (int wm = 0, n; wm < (w.ct == 16 ? 2 : 4); ++wm, tiles |= 1u << n) {
          n = 0;
          for (int r = 0; r < w.rt; ++r) n += r * (w.ct == 16 ? 2 : 4) + wm < std::min(w.block_tiles, rt - rb * w.block_tiles);
        }
      printf("%d %d %d %d %d %d %u\n", rows, i, w.ct, w.rt, w.whole, p.P > 1, tiles);
    }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    d = tmp_path_factory.mktemp("plans")
    (d / "plans.cpp").write_text(PLANS)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "plans"), str(d / "plans.cpp")], check=True)

    def run(shape, passes, head):
        """The forms that passes (rows, mode) take: (epilogue, n-tiles, row tiles, whole, phases, row tiles of a wave); of the LM
        head (calls of several clients, if `head`), whose epilogue is the same code for any number of tiles, without the last."""
        r = subprocess.run([str(d / "plans"), *map(str, (shape.d_model, shape.q_dim, shape.kv_dim, shape.d_ffn, shape.vocab)),
                            *[str(v) for p in passes for v in p]], capture_output=True, text=True, check=True)
        got = {}
        for ln in r.stdout.splitlines():
            rows, product, ct, rt, whole, phases, tiles = map(int, ln.split())
            if product == 4:
                if head:
                    got.setdefault(("head", ct, rt, whole, phases), rows)
                continue
            for n in range(rt + 1):
                if tiles >> n & 1:
                    got.setdefault((("qkv", "resid", "swiglu", "resid")[product], ct, rt, whole, phases, n), rows)
        return got

    return run


def test_gpu_cases_reach_every_form_the_models_take(forms):
    from tests import test_gpu_prompt as prompt
    from tests import test_gpu_row_groups as groups
    from tests import test_gpu_wide_shapes as wide
    both = lambda rows: [(n, mode) for n in rows for mode in (0, 2)]
    reached = set()
    for shape in prompt.SHAPES:
        reached |= set(forms(shape, both(min(t - 1, 2048) for t in prompt.TOKENS), False))
    for shape in prompt.SHAPES[:3]:
        reached |= set(forms(shape, both(min(t, 2048) for t in prompt.TOKENS_BEHIND), False))
    for shape in groups.SHAPES:
        reached |= set(forms(shape, both(groups.ROWS), False))
    for shape, rows in wide.ROWS:
        reached |= set(forms(shape, both(rows), False))
    for shape in wide.HEADS:
        reached |= {f for f in forms(shape, [(n, 0) for n in wide.HEAD_ROWS], True) if f[0] == "head"}
    other = [I.ModelShape("3072", 1, 3072, 24, 8, 128, 8192, 32000), I.ModelShape("6144", 1, 6144, 48, 8, 128, 16384, 32000)]
    for shape in (I.LLAMA_1B, I.LLAMA_8B, I.LLAMA_13B, *other):
        taken = forms(shape, [(n, 0) for n in range(33, 2049)], True)
        assert len(taken) > 40
        missing = {f: rows for f, rows in taken.items() if f not in reached}
        assert not missing, f"{shape.name}: forms that no GPU test compares, and the first rows that take them: {missing}"


# Products whose walks are short: (model columns, query columns, KV columns, FFN), rows, epilogue, and what the shapes (n-tiles per
# workgroup, row tiles per wave), walking all of K, took on an MI355X (us; splits take longer).  The end of a large tile is what
# decides; a model of the time without it chose 16 x 4 in all of them but the QKV product of 1200 rows.
SHORT = [((1024, 1024, 512, 3072), 2047, "swiglu", {(8, 1): 66.4, (16, 2): 70.2, (8, 2): 71.2, (16, 4): 78.8, (16, 3): 88.4, (8, 3): 88.6}),
         ((1024, 1024, 512, 3072), 1200, "qkv", {(8, 1): 27.6, (16, 2): 28.2, (8, 2): 28.5, (8, 3): 35.6, (16, 3): 36.0, (16, 4): 43.2}),
         ((1536, 1536, 256, 9216), 1000, "swiglu", {(8, 1): 124.8, (8, 2): 140.8, (16, 2): 141.9, (16, 4): 144.6, (16, 3): 148.8, (8, 3): 148.9}),
         ((2560, 4096, 1024, 9728), 2047, "qkv", {(16, 2): 133.5, (8, 2): 134.6, (8, 1): 141.4, (16, 4): 154.6, (16, 3): 172.6, (8, 3): 176.6}),
         ((2560, 4096, 1024, 9728), 640, "swiglu", {(8, 2): 128.6, (16, 2): 130.7, (8, 1): 134.9, (16, 4): 141.1, (8, 3): 148.4, (16, 3): 151.4})]


@pytest.mark.parametrize("widths,rows,epilogue,us", SHORT)
def test_short_walks_take_one_of_the_fastest_shapes(forms, widths, rows, epilogue, us):
    d, q, kv, ffn = widths
    shape = I.ModelShape("short", 1, d, q // 64, kv // 64, 64, ffn, 32000)
    chosen = {f[1:4] for f in forms(shape, [(rows, 0)], False) if f[0] == epilogue}
    (ct, rt, whole), = chosen
    assert whole and us[ct, rt] <= 1.02 * min(us.values())
