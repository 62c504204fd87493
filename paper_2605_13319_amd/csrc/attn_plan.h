// How the attention of a pass is cut up, and how much memory its partial results take: plain host
// arithmetic, free of HIP, shared by the launchers and by the sizing of the scratch buffer.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <utility>

#include "../../include/pipesd.h"

namespace pipesd {

constexpr int kMaxRows = PIPESD_MAX_ROWS;  // rows of one client per pass (k + 1)
constexpr int kMaxPassRows = 256;          // rows of all clients that share a pass (bf16)
constexpr int kMaxPromptRows = 2048;       // rows of one client's prompt that share a pass (bf16)
constexpr int kPromptBlockRows = 128;      // rows of a prompt that attend as one client of the pass
constexpr int kMaxPassClients = 16;        // clients whose rows share one pass (each has at least 2 rows)
constexpr int kPartPad = 4;  // a partial row is [head_dim values, max, sum, 2 unused] so that rows stay 16-byte aligned

// streaming attention kernel (bf16 cache)
constexpr int kStreamWaves = 4;                // waves per workgroup: one per SIMD, so that two workgroups in different
                                               // phases (waiting for keys and values / multiplying) share a compute unit
constexpr int kStreamWgTokens = kStreamWaves * 32;  // tokens per workgroup and step
constexpr int kStreamMaxSteps = 64;            // steps of a split (a lane per step holds its block-table entries)
constexpr int kStreamMinSpan = 256;            // a client's context is cut into at most kStreamMaxSplits
constexpr int kStreamMaxSplits = 16;           // splits of 256 * 2^j tokens, j as small as that allows
constexpr int kPromptStep = 32;                // prompt kernel: tokens per step
constexpr int kAttnCounters = kMaxPassClients * 512;  // arrival counters

struct AttnClient {
  int32_t row_off, m, start_pos;  // the client's rows in the pass; position of its first row
  int32_t table_off;              // entries from KvView::table to the client's block table
  int32_t nsplit, part_off;       // splits of its context; floats from the partial buffer's start to the client's partials
  int32_t span, count_off;        // streaming kernel: tokens per split, the client's first arrival counter
};
struct AttnBatch {
  int32_t n;
  AttnClient c[kMaxPassClients];
};
struct PromptShares {
  int32_t n[kMaxPassClients];  // workgroups that share a client's spans
};

// the batch of a prompt's attention: its blocks of 128 rows, one "client" each
inline AttnBatch prompt_blocks(int rows, int start_pos) {
  AttnBatch b{};
  for (int r0 = 0; r0 < rows; r0 += kPromptBlockRows) {
    AttnClient& ac = b.c[b.n++];
    ac.row_off = r0;
    ac.m = std::min(kPromptBlockRows, rows - r0);
    ac.start_pos = start_pos + r0;
  }
  return b;
}
static_assert(kMaxPromptRows <= kMaxPassClients * kPromptBlockRows, "a prompt's blocks fit a batch");

inline int attn_query_tiles(int group, int m) { return (group * m + 15) / 16; }  // of the rows that share a KV head

// Splits wanted of a prompt block of m rows (33 .. 128) at a context of `total` tokens.  The query tiles
// alone give many workgroups, so the context is cut only as far as it takes for the block by itself to
// have about two workgroups per compute unit (by itself: its results do not depend on how many blocks
// of the prompt share the pass), and as far as a split's largest number of steps asks for.
inline long prompt_block_splits(int group, int n_kv_heads, int m, int64_t total, int n_cu) {
  const long groups = (long)n_kv_heads * ((attn_query_tiles(group, m) + 1) / 2);
  const long fit = (long)((total + kStreamMaxSteps * kStreamWgTokens - 1) / (kStreamMaxSteps * kStreamWgTokens));
  return std::max(fit, std::min((long)kStreamMaxSplits, 2L * n_cu / groups));
}

// Passes of at most kMaxRows rows per client, and prompts, whose blocks of up to kPromptBlockRows rows
// are the clients of the batch (`prompt`), take the streaming kernel (bf16 cache), or the prompt kernel with the
// same spans and the same results (attn_prompt_shares).  Fills span,
// nsplit, part_off and count_off of every client of `b` (row_off, m, start_pos, table_off given) and
// returns the query tiles per workgroup, or 0 if the pass does not fit (then the split kernels run);
// *part_floats = size of the partial buffer the launch needs.  A client's split depends on its own
// context only, so its results do not depend on who shares the pass.
inline int attn_stream_plan(int n_q_heads, int n_kv_heads, int head_dim, int n_cu, AttnBatch& b, bool prompt,
                            size_t* part_floats) {
  *part_floats = 0;
  if (b.n < 1 || b.n > kMaxPassClients || (head_dim != 128 && head_dim != 64)) return 0;
  const int group = n_q_heads / n_kv_heads;
  int max_m = 1;
  long tasks = 0;  // (kv head, split, query tile) over all clients
  for (int i = 0; i < b.n; ++i) {
    AttnClient& cl = b.c[i];
    if (cl.m > (prompt ? kPromptBlockRows : kMaxRows)) return 0;
    max_m = std::max(max_m, (int)cl.m);
    const int total = cl.start_pos + cl.m;
    cl.span = kStreamMinSpan;
    if (cl.m <= kMaxRows) {
      while ((total + cl.span - 1) / cl.span > kStreamMaxSplits) cl.span *= 2;
    } else {
      const long want = prompt_block_splits(group, n_kv_heads, cl.m, total, n_cu);
      const int steps = (total + kStreamMinSpan - 1) / kStreamMinSpan;
      cl.span = (int)((steps + want - 1) / want) * kStreamMinSpan;
    }
    cl.nsplit = (total + cl.span - 1) / cl.span;
    if (cl.span > kStreamMaxSteps * kStreamWgTokens || cl.nsplit > kStreamMaxSplits) return 0;  // (contexts beyond 131072 tokens)
    tasks += (long)n_kv_heads * cl.nsplit * attn_query_tiles(group, cl.m);
  }
  // two tiles per workgroup (keys and values read once for both) where a head group has exactly
  // two, or where single tiles would be more workgroups than two rounds of the device
  const int max_qt = attn_query_tiles(group, max_m);
  const int T = (max_qt == 2 || tasks > 2L * n_cu) ? 2 : 1;
  if ((long)n_kv_heads * ((max_qt + T - 1) / T) > kAttnCounters / kMaxPassClients) return 0;
  size_t floats = 0;
  for (int i = 0; i < b.n; ++i) {
    AttnClient& cl = b.c[i];
    if (floats > (size_t)INT32_MAX) return 0;
    cl.part_off = (int32_t)floats;
    cl.count_off = i * (kAttnCounters / kMaxPassClients);
    const int nz = (attn_query_tiles(group, cl.m) + T - 1) / T;  // (the client's own tiles: the kernel's layout)
    floats += (size_t)n_kv_heads * nz * cl.nsplit * T * 16 * (head_dim + kPartPad);
  }
  *part_floats = floats;
  return T;
}

// Several clients in the streaming kernel's launch, T query tiles per workgroup.  Items (client, tile group, split): the items of
// a client side by side, the clients whose workgroups take longest first, so that what a round of workgroups more has left is
// short.  Only what there is to do is launched: with a grid of splits x the tile groups of the
// largest client 42 % of the workgroups of the 16-client call had nothing to do, but each took half a compute unit until it had
// found that out, and a client was found by a chain of loads (75.3 -> 72.1 us a layer, the call 9235 -> 9155).  That grid ran the clients'
// first tile groups before the others; items in the order of the clients, a split's tile groups next to each other, left long
// workgroups for the last round: calls of 4 clients behind up to 8000 tokens, us, that grid / the clients' order / this one: 8B widths
// (8 layers) 1513 / 1523 / 1454, 3072 columns on 8 KV heads 1009 / 1041 / 975, 1B 1497 / 1479 / 1430; 16 behind up to 4000 2771 / 2596 /
// 2575, 1783 / 1648 / 1622 and 2377 / 2219 / 2181.
struct StreamItems {
  int32_t first[kMaxPassClients];  // of client i of `batch` (beyond the batch: the number of items)
  int32_t n;                       // all items
};
inline StreamItems attn_stream_items(int group, int T, AttnBatch& batch) {
  auto longest = [&](const AttnClient& c) {  // (a workgroup's steps, and how many tiles it multiplies in each)
    return std::min((long)c.span, (long)c.start_pos + c.m) * (1 + std::min(T, attn_query_tiles(group, c.m)));
  };
  for (int i = 1; i < batch.n; ++i)
    for (int j = i; j > 0 && longest(batch.c[j]) > longest(batch.c[j - 1]); --j) std::swap(batch.c[j], batch.c[j - 1]);
  StreamItems items{};
  for (int i = 0; i < kMaxPassClients; ++i) {
    items.first[i] = items.n;
    if (i < batch.n) items.n += batch.c[i].nsplit * ((attn_query_tiles(group, batch.c[i].m) + T - 1) / T);
  }
  return items;
}

// Which kernel takes a planned pass: 0 for the streaming kernel, else the prompt kernel, with `shares`->n[i] workgroups
// for (a KV head's four query tiles of) client i, each with spans of its own, and their sum returned.  Either way
// every row gets the same bits: the rule is about time.  The work is cut into about twice as many shares as the device
// holds workgroups (two per compute unit), none below 8 steps: 2047 rows at the 8B shape 117 us with one share per slot,
// 113 with two, 120 with four.
//
// The prompt kernel's workgroups are long (a wave walks all tokens of its spans), so it needs many of them, and
// its time goes by groups of four tiles, whether a last one is full or not.  Both kernels were timed at 14 shapes (1B, 8B and 13B;
// 16 to 128 query heads, 2 to 64 KV heads, either head size), 33 to 900 rows behind 0 to 7000 tokens.  Of 2995 passes that the rule
// below gives to the prompt kernel 4 are slower by more than 2.5 % of the call (48 heads of 64 on 8 KV heads, 270 and 290 rows
// behind 4000 to 7000 tokens: 3 to 12 %).  It also keeps passes back that would gain, at the three models none more than
// 5 %.  Changes of a layer's attention, streaming -> prompt kernel, on the two sides of its lines:
//  * workgroups up to half a compute unit each: 16 heads of 128, 200 rows behind 300 tokens (128 workgroups) + 3.7 us, 289
//    rows (96) + 4.6; 8B shape, 128 rows behind 300 (128) - 1.2, 129 rows (144) - 5.3;
//  * contexts of one span, one each: 64 heads of 64, 127 to 240 rows alone (128 to 240) + 1.7 to 2.6, 256 rows (256) + 1.0,
//    heads of 128, 128 heads (256) 0 to - 3;
//  * walks of 32 and more steps, one and five eighths each, and 96 groups: 64 heads of 64 on 4 KV heads, 129 rows behind 3000 (292
//    workgroups, 56 steps) + 9.4, 48 heads of 128, 129 behind 1900 (256, 32) + 7.2, 1B shape, 150 behind 5000 (432, 48, 80 groups)
//    + 10.8; 8B shape, 200 rows behind 3000 (536, 32) - 7.2, 256 behind 6000 (512, 56) - 25;
//  * head size 64, groups of less than 84 % tiles: 64 KV heads, 129 rows behind 900 and 6000 (75 %) + 6.9 and + 10.7.
inline int attn_prompt_shares(int group, int n_kv_heads, int head_dim, int n_cu, const AttnBatch& b, PromptShares* shares) {
  int max_m = 0, most = 0;
  long tiles = 0, groups = 0, work = 0;  // query tiles; groups of four of them; steps of all groups
  auto steps_of = [](const AttnClient& cl) { return (cl.start_pos + cl.m + kPromptStep - 1) / kPromptStep; };
  auto groups_of = [&](const AttnClient& cl) { return (long)n_kv_heads * ((attn_query_tiles(group, cl.m) + kStreamWaves - 1) / kStreamWaves); };
  for (int i = 0; i < b.n; ++i) {
    max_m = std::max(max_m, (int)b.c[i].m);
    most = std::max(most, (int)(b.c[i].start_pos + b.c[i].m));
    tiles += (long)n_kv_heads * attn_query_tiles(group, b.c[i].m);
    groups += groups_of(b.c[i]);
    work += groups_of(b.c[i]) * steps_of(b.c[i]);
  }
  if (max_m <= kMaxRows) return 0;  // (rounds of clients, prompts of a few rows)
  if (groups < 64 || (head_dim == 64 && 25 * tiles < 84 * groups)) return 0;
  const long share_steps = std::max(8L, work / (4L * n_cu));
  long sum = 0, workgroups = 0, walk = 0;  // walk: the most steps of a workgroup
  for (int i = 0; i < b.n; ++i) {
    const AttnClient& cl = b.c[i];
    const long n = std::min((long)cl.nsplit, (steps_of(cl) + share_steps - 1) / share_steps);
    shares->n[i] = (int)n;
    sum += n;
    workgroups += groups_of(cl) * n;
    walk = std::max(walk, std::min((long)steps_of(cl), (cl.nsplit + n - 1) / n * (cl.span / kPromptStep)));
  }
  const long eighths = 8 * workgroups / n_cu;  // of a workgroup per compute unit
  if (2 * workgroups <= n_cu || (most <= kStreamMinSpan && eighths < 8)) return 0;
  if (walk >= 32 && (groups < 96 || eighths < 13)) return 0;
  return (int)sum;
}

// Floats of attention partials that no pass over a pool of `pool_tokens` cached tokens exceeds, but for
// the ones named below.
//  * NAV passes: up to `clients` clients of up to `rows` rows, contexts of at most the pool together, split
//    no finer than `chunk` tokens, a head group's rows rounded up to whole pairs of 16-row tiles.  (An
//    fp32 model's prompt blocks are such passes, of one client.)
//  * Prompts of a bf16 model on the streaming kernel: up to 16 blocks, all of 128 rows but the last, which
//    is cut finer the fewer rows it has: the worst number of rows is looked for.
// Not covered: prompt passes the streaming plan declines (a context beyond 131072 tokens, more than 128
// query heads) and the partials per layer of the all-layers kernel.  They would make every pool pay for
// what few callers do: 4 times the floats for the former.
inline size_t attn_scratch_floats(int n_q_heads, int n_kv_heads, int head_dim, int n_cu, int clients, int rows, int chunk,
                                  bool stream_prompts, int64_t pool_tokens) {
  const int group = n_q_heads / n_kv_heads;
  const size_t row = (size_t)n_kv_heads * (head_dim + kPartPad);
  const size_t nav = (size_t)(pool_tokens / chunk + clients) * (size_t)(group * rows + 31) * row;
  if (!stream_prompts) return nav;
  const int64_t steps = (pool_tokens + kStreamMinSpan - 1) / kStreamMinSpan;
  auto block_rows = [&](int m) {  // (rows, padded) x splits of a block of m rows behind the longest context
    const long want = m <= kMaxRows ? kStreamMaxSplits : prompt_block_splits(group, n_kv_heads, m, pool_tokens, n_cu);
    const int64_t splits = std::min((int64_t)std::min(want, (long)kStreamMaxSplits), steps);
    return (size_t)splits * ((attn_query_tiles(group, m) + 1) / 2 * 2) * 16;
  };
  size_t last = 0;
  for (int m = 1; m <= kPromptBlockRows; ++m) last = std::max(last, block_rows(m));
  const int64_t blocks = (std::min(pool_tokens, (int64_t)kMaxPromptRows) + kPromptBlockRows - 1) / kPromptBlockRows;
  return std::max(nav, ((size_t)(blocks - 1) * block_rows(kPromptBlockRows) + last) * row);
}

}  // namespace pipesd
