"""The attention scratch that a cache pool is given at its creation holds the partials of every pass over
it: the planner of the streaming attention swept over rows, starts and pool sizes on the host."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_13319_amd", "csrc")

SWEEP = r"""
#include <stdio.h>
#include <stdlib.h>
#include "attn_plan.h"
using namespace pipesd;
static long checked = 0;
static bool check(int nq, int nkv, int hd, int n_cu, AttnBatch b, bool prompt, long pool, const char* what) {
  size_t need = 0;
  const int T = attn_stream_plan(nq, nkv, hd, n_cu, b, prompt, &need);
  if (T == 0) return true;  // (declined: the split kernels)
  const size_t have = attn_scratch_floats(nq, nkv, hd, n_cu, kMaxPassClients, kMaxRows, 256, true, pool);
  // the kernel's layout: client after client, [kv head][own tile groups][split][T][16][head_dim + pad]
  size_t end = 0;
  for (int i = 0; i < b.n; ++i) {
    const AttnClient& c = b.c[i];
    if ((size_t)c.part_off != end || (end * 4) % 128) { printf("%s: client %d at %d, not %zu\n", what, i, c.part_off, end); return false; }
    end += (size_t)nkv * ((((nq / nkv) * c.m + 15) / 16 + T - 1) / T) * c.nsplit * T * 16 * (hd + 4);
  }
  ++checked;
  if (end <= need && need <= have) return true;
  printf("%s: heads %d/%d x %d, pool %ld: used %zu, planned %zu, there %zu (first client: %d rows behind %d, n = %d)\n", what, nq, nkv, hd,
         pool, end, need, have, b.c[0].m, b.c[0].start_pos, b.n);
  return false;
}
int main(int argc, char** argv) {
  const int nq = atoi(argv[1]), nkv = atoi(argv[2]), hd = atoi(argv[3]), n_cu = atoi(argv[4]);
  unsigned seed = 12345;
  auto rnd = [&](long n) { seed = seed * 1664525u + 1013904223u; return (long)((seed >> 8) % (unsigned long)n); };
  for (long pool : {16L, 112L, 1024L, 2048L, 2064L, 4096L, 10000L, 33008L, 131072L, 262144L}) {
    for (long rows = 33; rows <= 2048 && rows <= pool; ++rows)
      for (int s = 0; s < 5; ++s) {
        const long room = pool - rows, start = s == 0 ? 0 : s == 1 ? room : s == 2 ? room / 2 : rnd(room + 1);
        if (!check(nq, nkv, hd, n_cu, prompt_blocks((int)rows, (int)start), true, pool, "prompt")) return 1;
      }
    for (int t = 0; t < 2000; ++t) {  // rounds of 1 .. 16 clients whose blocks of 16 tokens share the pool
      AttnBatch b{};
      long left = pool / 16, rows = 0;
      const int n = 1 + (int)rnd(16);
      for (int i = 0; i < n && left > 0; ++i) {
        const long m = 1 + rnd(32), most = left - (n - 1 - i) > 0 ? left - (n - 1 - i) : 1;
        const long blocks = i == n - 1 ? left : 1 + rnd(most);
        if (blocks * 16 < m || rows + m > kMaxPassRows) continue;
        AttnClient& c = b.c[b.n++];
        c.row_off = (int)rows;
        c.m = (int)m;
        c.start_pos = (int)(blocks * 16 - m);
        rows += m;
        left -= blocks;
      }
      if (b.n > 0 && !check(nq, nkv, hd, n_cu, b, false, pool, "round")) return 1;
    }
  }
  printf("%ld plans\n", checked);
  return checked > 10000 ? 0 : 1;
}
"""


@pytest.fixture(scope="module")
def sweep(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    d = tmp_path_factory.mktemp("plan")
    (d / "sweep.cpp").write_text(SWEEP)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "sweep"), str(d / "sweep.cpp")], check=True)
    return str(d / "sweep")


# head groups of 1, 4, 8, 16 and 128 heads, both head sizes; the largest number of heads the kernel takes
@pytest.mark.parametrize("heads", [(32, 8, 128), (32, 8, 64), (40, 40, 128), (8, 2, 64), (16, 1, 128), (64, 8, 64), (128, 128, 64),
                                   (128, 8, 64), (128, 1, 64)])
@pytest.mark.parametrize("n_cu", [256, 64])
def test_scratch_of_a_pool_holds_every_pass(sweep, heads, n_cu):
    r = subprocess.run([sweep, *map(str, heads), str(n_cu)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout


ITEMS = r"""
#include <stdio.h>
#include <stdlib.h>
#include "attn_plan.h"
using namespace pipesd;
static unsigned seed = 4321;
static long rnd(long n) { seed = seed * 1664525u + 1013904223u; return (long)((seed >> 8) % (unsigned long)n); }
int main() {
  const int heads[][3] = {{32, 8, 128}, {24, 8, 128}, {32, 8, 64}, {40, 40, 128}, {128, 1, 64}, {16, 16, 64}};
  int checked = 0;
  for (int t = 0; t < 6000; ++t) {
    const int* h = heads[t % 6], group = h[0] / h[1];
    AttnBatch b{};
    b.n = 2 + (int)rnd(15);
    int rows = 0;
    for (int i = 0; i < b.n; ++i) {
      b.c[i].row_off = rows;
      rows += b.c[i].m = 1 + (int)rnd(17);
      b.c[i].start_pos = (int)rnd(rnd(20000) + 1);
    }
    size_t floats = 0;
    const int T = attn_stream_plan(h[0], h[1], h[2], 256, b, false, &floats);
    if (T == 0) continue;
    AttnBatch o = b;
    const StreamItems items = attn_stream_items(group, T, o);
    // every (client, tile group, split) of the plan once, found as the kernel finds it
    static unsigned char seen[kMaxPassClients][2048][kStreamMaxSplits];
    for (auto& c : seen) for (auto& z : c) for (auto& s : z) s = 0;
    long last = -1;
    for (int item = 0; item < items.n; ++item) {
      int ci = 0;
      for (int i = 1; i < kMaxPassClients; ++i) ci += item >= items.first[i] ? 1 : 0;
      if (ci >= o.n) return 1;
      const AttnClient& c = o.c[ci];
      const int z = (item - items.first[ci]) / c.nsplit, s = item - items.first[ci] - z * c.nsplit;
      int was = -1;
      for (int i = 0; i < b.n; ++i) if (b.c[i].row_off == c.row_off) was = i;
      if (was < 0 || z * T >= attn_query_tiles(group, c.m) || c.m != b.c[was].m || c.start_pos != b.c[was].start_pos || c.part_off != b.c[was].part_off ||
          c.count_off != b.c[was].count_off || c.span != b.c[was].span || seen[was][z][s]++) return 2;
      // no client's workgroups are longer than those of the clients before it
      const long steps = std::min((long)c.span, (long)c.start_pos + c.m) * (1 + std::min(T, attn_query_tiles(group, c.m)));
      if (last >= 0 && steps > last) return 3;
      last = steps;
    }
    long all = 0, found = items.n;
    for (int i = 0; i < b.n; ++i) all += (long)b.c[i].nsplit * ((attn_query_tiles(group, b.c[i].m) + T - 1) / T);
    if (all != found || all > 65535) return 4;  // (a grid's limit)
    ++checked;
  }
  return checked > 3000 ? 0 : 5;
}
"""


def test_items_of_several_clients_are_each_there_once_the_longest_first(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    (tmp_path / "items.cpp").write_text(ITEMS)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", str(tmp_path / "items"), str(tmp_path / "items.cpp")], check=True)
    assert subprocess.run([str(tmp_path / "items")], timeout=120).returncode == 0


ROUTES = r"""
#include <stdio.h>
#include <stdlib.h>
#include "attn_plan.h"
using namespace pipesd;
// a prompt pass per line of arguments (rows, first position): 0 / 1 (prompt kernel), then per block rows:spans:tokens per span:workgroups
int main(int argc, char** argv) {
  const int nq = atoi(argv[1]), nkv = atoi(argv[2]), hd = atoi(argv[3]);
  for (int i = 4; i + 1 < argc; i += 2) {
    AttnBatch b = prompt_blocks(atoi(argv[i]), atoi(argv[i + 1]));
    size_t floats = 0;
    PromptShares s{};
    if (attn_stream_plan(nq, nkv, hd, 256, b, true, &floats) == 0) return 1;
    const int n = attn_prompt_shares(nq / nkv, nkv, hd, 256, b, &s);
    int sum = 0;
    printf("%d", n > 0);
    for (int j = 0; j < b.n; ++j) {
      printf(" %d:%d:%d:%d", b.c[j].m, b.c[j].nsplit, b.c[j].span, n > 0 ? s.n[j] : 0);
      sum += s.n[j];
      if (n > 0 && (s.n[j] < 1 || s.n[j] > b.c[j].nsplit || b.c[j].span % (4 * kPromptStep) != 0)) return 2;
    }
    if (n > 0 && sum != n) return 3;
    printf("\n");
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    d = tmp_path_factory.mktemp("routes")
    (d / "routes.cpp").write_text(ROUTES)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "routes"), str(d / "routes.cpp")], check=True)

    def run(shape, passes):
        """Per (rows, first position): whether the prompt kernel takes it, and its blocks (rows, spans, tokens per span, workgroups)."""
        r = subprocess.run([str(d / "routes"), str(shape.n_q_heads), str(shape.n_kv_heads), str(shape.head_dim),
                            *[str(v) for p in passes for v in p]], capture_output=True, text=True, check=True)
        lines = [ln.split() for ln in r.stdout.splitlines()]
        return [(ln[0] == "1", [tuple(map(int, blk.split(":"))) for blk in ln[1:]]) for ln in lines]

    return run


def test_the_gpu_cases_of_prompt_attention_take_the_kernels_they_are_meant_for(routes):
    from tests import test_gpu_prompt_attention as t

    def passes(cached, sizes):  # (rows, first position) of the calls
        got, length = [], cached
        for n in sizes:
            got.append((n - (1 if length == 0 else 0), max(0, length - 1)))
            length += n
        return got

    for shape in t.BIG:
        for tokens in t.SHORT + [257, 300]:
            assert routes(shape, passes(0, [tokens]))[0][0], (shape.name, tokens)
            assert not any(p for p, _ in routes(shape, passes(0, t.in_blocks(0, tokens, 32))))
    for shape in t.SHAPES:
        assert [r[0] for r in routes(shape, [(rows, 0) for rows in (128, 215, 299, 2048)])] == [False, False, shape.head_dim == 128, True]
    seen = {"spans of a lone workgroup": 0, "spans of several": 0, "most spans": 0, "longest walk": 0, "span": 0, "ragged": 0}
    for shape in t.SMALL:
        for cached, tokens in t.LONG:
            first_pass = min(tokens, 2048 + (cached == 0))
            taken, blocks = routes(shape, passes(cached, [first_pass]))[0]
            assert taken, (shape.name, cached, tokens)
            assert not any(p for p, _ in routes(shape, passes(cached, t.in_blocks(cached, tokens, 128))))
            for rows, spans, span, workgroups in blocks:
                if workgroups == 1:
                    seen["spans of a lone workgroup"] = max(seen["spans of a lone workgroup"], spans)
                elif workgroups < spans:
                    seen["spans of several"] = max(seen["spans of several"], spans)
                seen["most spans"] = max(seen["most spans"], spans)
                seen["longest walk"] = max(seen["longest walk"], spans * span // (32 * workgroups))
                seen["span"] = max(seen["span"], span)
                seen["ragged"] += rows % 128 != 0
    assert seen["spans of a lone workgroup"] >= 3 and seen["spans of several"] >= 4 and seen["most spans"] >= 10, seen
    assert seen["longest walk"] > 64 and seen["span"] > 256 and seen["ragged"] > 0, seen
    print(seen)


def test_prompt_attention_goes_where_it_was_measured_faster(routes):
    """Passes on both sides of the rule's lines: (query heads, KV heads, head size), (rows, first position), and whether the prompt
    kernel, the faster one there, takes them."""
    from paper_2605_13319_amd import inputs as I
    cases = [((32, 8, 128), (2047, 0), True), ((32, 8, 128), (333, 999), True), ((32, 8, 128), (128, 0), False),
             ((32, 8, 128), (129, 299), True), ((32, 8, 128), (128, 299), False),  # workgroups: half a compute unit each
             ((32, 8, 128), (255, 0), False), ((128, 16, 128), (128, 0), True),    # contexts of one span
             ((64, 4, 64), (129, 2999), False), ((48, 8, 128), (129, 1899), False), ((128, 8, 64), (129, 1899), False),  # long walks
             ((64, 8, 128), (97, 5999), False), ((32, 8, 64), (150, 4999), False), ((32, 8, 128), (200, 2999), True), ((32, 8, 128), (256, 5999), True),
             ((32, 8, 64), (256, 5999), True), ((40, 40, 128), (200, 5999), True),
             ((64, 64, 64), (129, 899), False), ((64, 64, 64), (129, 5999), False), ((64, 64, 64), (256, 899), True)]  # groups not full
    for (n_q, n_kv, hd), where, prompt in cases:
        shape = I.ModelShape("route", 2, 512, n_q, n_kv, hd, 512, 300)
        assert routes(shape, [where])[0][0] == prompt, (n_q, n_kv, hd, where)
