// How the attention of a pass is cut up, and how much memory its partial results take: plain host
// arithmetic, free of HIP, shared by the launchers and by the sizing of the scratch buffer.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

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
constexpr int kPromptMinSpan = 256;            // a block's context is cut into spans of at least this many
constexpr int kPromptFewTiles = 128, kPromptFewTokens = 2048;  // blocks the streaming kernel keeps: fewer tiles, up to as many tokens
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

// Rows of one client, or a block of a prompt, that the streaming kernel takes: as many as a round can have, and
// blocks that would leave the prompt kernel with few workgroups of many steps: fewer than 128 query tiles (32
// workgroups) behind up to 2048 tokens, or less than a full block at a context of 128 tokens, which the streaming
// kernel's four waves see in one step.  8B shape, microseconds on the streaming / the prompt kernel: 48 rows behind 1,
// 128, 300 and 900 tokens 5.7 / 6.8, 8.2 / 9.4, 11.2 / 13.2, 14.6 / 18.0; 128 rows behind 1, 128, 300 and 900 6.2 / 7.7,
// 15.0 / 11.0, 15.5 / 15.0, 27 / 28; 300 rows behind 1, 64 and 900 16 / 13, 22 / 15, 48 / 36.  (Both kinds of a prompt's blocks
// share a launch.)
inline bool attn_few_rows(int group, int n_kv_heads, int m, int64_t total) {
  return m <= kMaxRows || (m < kPromptBlockRows && total <= kPromptBlockRows) ||
         (total <= kPromptFewTokens && n_kv_heads * attn_query_tiles(group, m) < kPromptFewTiles);
}

// Splits wanted of another block at a context of `total` tokens: by the block alone (its results do not depend on
// how many blocks of the prompt share the pass), spans of 2048 tokens for a full block, of 8 per row for a
// last one, and no more than leave a workgroup per pair of tiles two of a compute unit (the partials' memory).  A
// split costs its partials' way through memory and their merge, about 6 us: 2047 rows at the 8B shape 85 us with spans
// of 2048 tokens, 101 with 1024, 124 with 512; 128 rows behind 2900 tokens 41, 36, 38.
inline long prompt_block_splits(int group, int n_kv_heads, int m, int64_t total, int n_cu) {
  const long span = m == kPromptBlockRows ? 2048 : std::max(kPromptMinSpan, 8 * m);
  const long most = 2L * n_cu / (n_kv_heads * ((attn_query_tiles(group, m) + 1) / 2));
  return std::max(1L, std::min({(long)kStreamMaxSplits, most, (long)((total + span - 1) / span)}));
}

// Passes of at most kMaxRows rows per client, and prompts, whose blocks of up to kPromptBlockRows rows
// are the clients of the batch (`prompt`), take the streaming kernel (bf16 cache).  Fills span,
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
  bool blocks = false;
  for (int i = 0; i < b.n; ++i) {
    AttnClient& cl = b.c[i];
    if (cl.m > (prompt ? kPromptBlockRows : kMaxRows)) return 0;
    max_m = std::max(max_m, (int)cl.m);
    const int total = cl.start_pos + cl.m;
    cl.span = kStreamMinSpan;
    if (attn_few_rows(group, n_kv_heads, cl.m, total)) {
      while ((total + cl.span - 1) / cl.span > kStreamMaxSplits) cl.span *= 2;
    } else {
      blocks = true;
      const long want = prompt_block_splits(group, n_kv_heads, cl.m, total, n_cu);
      cl.span = (int)((total + want * kPromptStep - 1) / (want * kPromptStep)) * kPromptStep;
    }
    cl.nsplit = (total + cl.span - 1) / cl.span;
    if (total > kStreamMaxSplits * kStreamMaxSteps * kStreamWgTokens) return 0;  // (contexts beyond 131072 tokens)
    tasks += (long)n_kv_heads * cl.nsplit * attn_query_tiles(group, cl.m);
  }
  // two tiles per workgroup (keys and values read once for both) where a head group has exactly
  // two, or where single tiles would be more workgroups than two rounds of the device
  // (one where a prompt's last block shares a launch with blocks of the prompt kernel)
  const int max_qt = attn_query_tiles(group, max_m);
  const int T = !blocks && (max_qt == 2 || tasks > 2L * n_cu) ? 2 : 1;
  size_t floats = 0;
  for (int i = 0; i < b.n; ++i) {
    AttnClient& cl = b.c[i];
    if (floats > (size_t)INT32_MAX) return 0;
    const int qt = attn_query_tiles(group, cl.m), per_wg = attn_few_rows(group, n_kv_heads, cl.m, cl.start_pos + cl.m) ? T : kStreamWaves;
    if ((long)n_kv_heads * ((qt + per_wg - 1) / per_wg) > kAttnCounters / kMaxPassClients) return 0;
    cl.part_off = (int32_t)floats;
    cl.count_off = i * (kAttnCounters / kMaxPassClients);
    const int nz = (attn_query_tiles(group, cl.m) + T - 1) / T;  // (the client's own tiles: the kernel's layout)
    floats += (size_t)n_kv_heads * nz * cl.nsplit * T * 16 * (head_dim + kPartPad);
  }
  *part_floats = floats;
  return T;
}

// Floats of attention partials that no pass over a pool of `pool_tokens` cached tokens exceeds, but for
// the ones named below.
//  * NAV passes: up to `clients` clients of up to `rows` rows, contexts of at most the pool together, split
//    no finer than `chunk` tokens, a head group's rows rounded up to whole pairs of 16-row tiles.  (An
//    fp32 model's prompt blocks are such passes, of one client.)
//  * Prompts of a bf16 model on the prompt and streaming kernels: up to 16 blocks, all of 128 rows but the last, which
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
    // (behind the longest context, or behind the longest at which the streaming kernel takes as many rows)
    const long want = m <= kMaxRows ? kStreamMaxSplits
                                    : std::max(prompt_block_splits(group, n_kv_heads, m, pool_tokens, n_cu),
                                               n_kv_heads * attn_query_tiles(group, m) < kPromptFewTiles ? (long)(kPromptFewTokens / kStreamMinSpan) : 1L);
    const int64_t splits = std::min((int64_t)std::min(want, (long)kStreamMaxSplits), steps);
    return (size_t)splits * ((attn_query_tiles(group, m) + 1) / 2 * 2) * 16;
  };
  size_t last = 0;
  for (int m = 1; m <= kPromptBlockRows; ++m) last = std::max(last, block_rows(m));
  const int64_t blocks = (std::min(pool_tokens, (int64_t)kMaxPromptRows) + kPromptBlockRows - 1) / kPromptBlockRows;
  return std::max(nav, ((size_t)(blocks - 1) * block_rows(kPromptBlockRows) + last) * row);
}

}  // namespace pipesd
