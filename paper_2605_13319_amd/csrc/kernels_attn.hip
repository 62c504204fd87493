// Grouped-query attention of the m = k + 1 causal rows of a pass over the paged KV cache.
// (Masked self-attention of a decoder-only layer, Sec. 2.1; row r sees key positions 0..pos_r.)
//
// Split over the context: workgroup (kv_head, split) handles `chunk` consecutive tokens for every
// query row of the query heads that share the KV head, producing an un-normalised partial
// (max, sum, o); a second kernel merges the splits in a fixed order, so results do not depend on
// scheduling.
#include <algorithm>
#include <type_traits>

#include "device_attn.h"
#include "device_dma.h"
#include "lds_limit.h"

namespace pipesd {

constexpr int kAttnThreads = 256;
constexpr int kAttnChunkMax = 32;

template <typename T>
__global__ __launch_bounds__(kAttnThreads) void attn_partial_kernel(const float* __restrict__ q, KvView kv, int layer,
                                                                    int m, int start_pos, int n_q_heads, int chunk,
                                                                    int nsplit, float* __restrict__ part) {
  extern __shared__ float lds[];
  const int h = kv.head_dim;
  const int hp = h + 1;
  float* ks = lds;                          // [chunk][h+1]
  float* vs = ks + kAttnChunkMax * hp;      // [chunk][h+1]
  float* qs = vs + kAttnChunkMax * hp;      // [m][h]
  float* ps = qs + kMaxRows * h;            // [m][chunk]
  const int kvh = blockIdx.x, split = blockIdx.y;
  const int group = n_q_heads / kv.n_kv_heads;
  const int total = start_pos + m;          // keys visible to the last row
  const int t0 = split * chunk;
  const int nt = min(chunk, total - t0);
  const int tid = threadIdx.x;
  const T* pool = (const T*)kv.pool;
  const float scale = 1.0f / sqrtf((float)h);

  for (int i = tid; i < nt * h; i += kAttnThreads) {
    const int t = i / h, e = i % h;
    ks[t * hp + e] = load_elem(pool, k_index(kv, layer, t0 + t, kvh, e));
  }
  for (int i = tid; i < nt * h; i += kAttnThreads) {
    const int e = i / nt, t = i % nt;  // the value block keeps tokens contiguous per element
    vs[t * hp + e] = load_elem(pool, v_index(kv, layer, t0 + t, kvh, e));
  }

  for (int gq = 0; gq < group; ++gq) {
    const int head = kvh * group + gq;
    __syncthreads();
    for (int i = tid; i < m * h; i += kAttnThreads) {
      const int r = i / h, e = i % h;
      qs[i] = q[((size_t)r * n_q_heads + head) * h + e];
    }
    __syncthreads();
    // scores
    for (int i = tid; i < m * chunk; i += kAttnThreads) {
      const int r = i / chunk, t = i % chunk;
      float s = -INFINITY;
      if (t < nt && t0 + t <= start_pos + r) {
        float acc = 0.f;
        for (int e = 0; e < h; ++e) acc = fmaf(qs[r * h + e], ks[t * hp + e], acc);
        s = acc * scale;
      }
      ps[i] = s;
    }
    __syncthreads();
    // per row: max, exp, sum (one thread per row; rows and chunk are small)
    if (tid < m) {
      float mx = -INFINITY;
      for (int t = 0; t < chunk; ++t) mx = fmaxf(mx, ps[tid * chunk + t]);
      float l = 0.f;
      for (int t = 0; t < chunk; ++t) {
        const float s = ps[tid * chunk + t];
        const float p = (s == -INFINITY) ? 0.f : expf(s - mx);
        ps[tid * chunk + t] = p;
        l += p;
      }
      float* o = part + (((size_t)head * m + tid) * nsplit + split) * (h + kPartPad);
      o[h] = mx;
      o[h + 1] = l;
    }
    __syncthreads();
    // o = P V
    for (int i = tid; i < m * h; i += kAttnThreads) {
      const int r = i / h, e = i % h;
      float acc = 0.f;
      for (int t = 0; t < nt; ++t) acc = fmaf(ps[r * chunk + t], vs[t * hp + e], acc);
      part[(((size_t)head * m + r) * nsplit + split) * (h + kPartPad) + e] = acc;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// bf16 cache: the same computation on the matrix cores (device code in device_attn.h)
// ------------------------------------------------------------------------------------------------
// grid = (kv heads, splits of all clients of the pass one client after the other, query tiles of the
// largest client / qpw); a workgroup takes qpw query tiles (MULTI) or one
template <int HD, bool MULTI>
__global__ __launch_bounds__(kAttnWaves * 64) void attn_mfma_kernel(const float* q, KvView kv, int layer, int n_q_heads,
                                                                    AttnBatch batch, float* part, int qpw,
                                                                    const int32_t* gate) {
  extern __shared__ float lds[];
  if (gate != nullptr && *gate == 0) return;  // (uniform: a round of a chain that does not run)
  const int kvh = blockIdx.x;
  int ci = 0, split = blockIdx.y;
  while (ci + 1 < batch.n && split >= batch.c[ci].nsplit) split -= batch.c[ci++].nsplit;
  const AttnClient c = batch.c[ci];
  const int nqt = (n_q_heads / kv.n_kv_heads * c.m + 15) / 16, qt0 = (int)blockIdx.z * qpw;
  if (split >= c.nsplit || qt0 >= nqt) return;  // whole workgroup
  kv.table += c.table_off;
  attn_task<HD, false, MULTI>(q + (size_t)c.row_off * n_q_heads * HD, kv, layer, c.m, c.start_pos, n_q_heads,
                              c.nsplit, part + c.part_off, kvh, split, qt0, min(nqt, qt0 + qpw), lds);
}

// ------------------------------------------------------------------------------------------------
// bf16 cache, passes of few rows per client (the NAV pass itself) and prompt passes of few blocks
// (attn_prompt_shares): one workgroup walks a whole split of the context
// ------------------------------------------------------------------------------------------------
// Workgroup (kv head, split of a client's context, T query tiles) of four waves: wave w takes tokens
// span0 + it*128 + w*32 .. + 31 in step it and keeps a running (max, sum, O) per query tile in
// registers.  A step's keys are requested one step ahead, into registers.  So are its values for
// T = 1; for T = 2 (twice the running state, no registers left for that) the values of the next
// step are copied from memory straight into an LDS buffer of the wave's own (the LDS its state goes
// to in the merge) as soon as the wave has read the current step's out of it, and travel during the
// rest of the step and the next step's scores.  After the last step the four waves' states are
// merged through LDS, waves in index order.  A client whose
// context is one split gets its normalised rows written straight in the packed form the O
// projection reads.  Otherwise the workgroup writes its partial through to memory and counts
// itself in; the workgroup that arrives last merges the splits, in index order, and writes the
// packed rows: no second launch.  The queries of the workgroup's tiles sit in LDS in operand order
// (hi and lo halves), read again in every step.  What a row's result is depends on the client's own
// context and rows only, never on the other clients of the pass, on T or on which workgroup came last.
//
// Partials: per (client, kv head, tile group) [split][T tiles][16 rows][HD + 4] floats, each
// [split] block a whole number of 128-byte lines, so no cache line holds partials of two groups:
// the merging workgroup reads lines nobody on its compute unit has touched during this kernel,
// after every writer has drained its write-through stores and then incremented the counter.
constexpr size_t stream_lds_floats(int hd) { return (size_t)kStreamWaves * 16 * (hd + 4) + 2 * kStreamWaves * 16; }
template <int HD>
constexpr size_t stream_lds_bytes(int T) {
  return stream_lds_floats(HD) * sizeof(float) + (size_t)T * (HD / 32) * 2 * 64 * 16 + 16;
}

// (grid: kv heads, and of several clients' items (attn_stream_items), of one client's splits, tile groups: finding its one
// item took 0.5 to 0.9 us)
template <int HD, int T>
__global__ __launch_bounds__(kStreamWaves * 64, 2) void attn_stream_kernel(const float* q, KvView kv, int layer, int n_q_heads,
                                                                      AttnBatch batch, StreamItems items, float* part,
                                                                      uint4* outp, int act_tiles, const int32_t* gate,
                                                                      unsigned* counters) {
  extern __shared__ float lds[];
  if (gate != nullptr && *gate == 0) return;  // (uniform: a round of a chain that does not run)
  constexpr int KSQ = HD / 32, HT = HD / 16, ROW = HD + 4;
  const int kvh = blockIdx.x;
  int ci = 0, split = blockIdx.y, zt = blockIdx.z;
  if (batch.n > 1) {
    const int item = blockIdx.y;
#pragma unroll
    for (int i = 1; i < kMaxPassClients; ++i) ci += item >= items.first[i] ? 1 : 0;
    const int ns = batch.c[ci].nsplit;
    zt = (item - items.first[ci]) / ns;
    split = item - items.first[ci] - zt * ns;
  }
  const AttnClient cl = batch.c[ci];
  const int group = n_q_heads / kv.n_kv_heads, m = cl.m, R = group * m;
  const int nqt = (R + 15) / 16, nz = (nqt + T - 1) / T, qt0 = zt * T;
  float(*o_lds)[16][ROW] = (float(*)[16][ROW])lds;
  float(*m_lds)[16] = (float(*)[16])(lds + (size_t)kStreamWaves * 16 * ROW);
  float(*l_lds)[16] = m_lds + kStreamWaves;
  au32x4* q_lds = (au32x4*)(lds + stream_lds_floats(HD));  // [T][KSQ][hi, lo][64 lanes]
  int* last_lds = (int*)(q_lds + T * KSQ * 2 * 64);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int total = cl.start_pos + m;
  const int span0 = split * cl.span, span1 = min(total, span0 + cl.span);
  const int nsteps = (span1 - span0 + kStreamWgTokens - 1) / kStreamWgTokens;
  const uint16_t* pool = (const uint16_t*)kv.pool;
  const int32_t* table = kv.table + cl.table_off;
  const float scale = 1.0f / sqrtf((float)HD);
  const float m_rinv = __builtin_amdgcn_rcpf((float)m);
  const int qd = n_q_heads * HD;

  // ---- queries of the T tiles: global (row = [qd hi halves][qd lo halves]) -> LDS in operand order ----
  constexpr int QCH = 16 * (HD / 8) * 2;  // 16-byte pieces per tile
  constexpr int QPT = (QCH + kStreamWaves * 64 - 1) / (kStreamWaves * 64);  // pieces per thread and tile
  au32x4 qreg[T][QPT];
  {
    const uint16_t* q16 = (const uint16_t*)q + (size_t)cl.row_off * 2 * qd;
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
      const int piece = tid + i * kStreamWaves * 64;
      const int hl = piece / (16 * (HD / 8)), rem = piece % (16 * (HD / 8)), qc = rem / (HD / 8), j = rem % (HD / 8);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int rr = (qt0 + t) * 16 + qc;  // rows beyond the head group read row 0 of the group (their results are dropped)
        const int gq = rr < R ? div_small(rr, m_rinv) : 0, r = rr < R ? rr - gq * m : 0;
        qreg[t][i] = piece < QCH ? *(const au32x4*)(q16 + (size_t)r * 2 * qd + hl * qd + (kvh * group + gq) * HD + j * 8)
                                 : au32x4{0u, 0u, 0u, 0u};
      }
    }
  }

  struct KRegs {
    au32x4 k[2][KSQ];
  };
  struct VRegs {
    au32x2 lo[HT], hi[HT];
  };
  // The block-table entries of this wave's tokens are read once, before the first step, and held in
  // registers: lane L has the two of step L (a split is at most 64 steps).  Looked up from memory
  // per request, every request would first wait for all loads before it, the step's keys and
  // values among them.
  int step_blk[2];
#pragma unroll
  for (int tt = 0; tt < 2; ++tt) {
    const int tb = span0 + lane * kStreamWgTokens + w * 32 + tt * 16;
    step_blk[tt] = table[tb < total ? tb / kBlockTokens : 0];
  }
  auto block_base = [&](int it, int tt) {
    const int blk = __builtin_amdgcn_readlane(step_blk[tt], it);
    return (int64_t)layer * kv.layer_stride + (int64_t)blk * kv.block_elems;
  };
  auto request_k = [&](KRegs& b, int it) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const int64_t base = block_base(it, tt);
#pragma unroll
      for (int s = 0; s < KSQ; ++s)
        b.k[tt][s] = *(const au32x4*)(pool + base + ((int64_t)kvh * kBlockTokens + c) * HD + s * 32 + g * 8);
    }
  };
  auto request_v = [&](VRegs& b, int it) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const int64_t base = block_base(it, tt);
#pragma unroll
      for (int j = 0; j < HT; ++j) {
        const au32x2 v = *(const au32x2*)(pool + base + kv.v_offset + ((int64_t)kvh * HD + j * 16 + c) * kBlockTokens + g * 4);
        if (tt == 0) b.lo[j] = v; else b.hi[j] = v;
      }
    }
  };

  // T = 2: the values of a step through LDS.  The wave's buffer holds the step's two blocks as they
  // are in memory ([element][16 tokens]); one load instruction copies 32 elements' rows (lane ->
  // element lane/2, tokens 8 (lane&1) .. +7).
  constexpr int NVL = 2 * (HD / 32);  // load instructions per step
  char* vbuf = (char*)lds + (size_t)w * 16 * ROW * sizeof(float);  // (= the wave's rows of o_lds)
  static_assert(2 * HD * kBlockTokens * 2 <= 16 * ROW * (int)sizeof(float), "a step's values fit the wave's merge rows");
  auto request_v_lds = [&](int it) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const int64_t base = block_base(it, tt);
#pragma unroll
      for (int qd32 = 0; qd32 < HD / 32; ++qd32) {
        const uint16_t* src = pool + base + kv.v_offset + ((int64_t)kvh * HD + qd32 * 32 + (lane >> 1)) * kBlockTokens + (lane & 1) * 8;
        lds_dma16(src, vbuf + (tt * (HD / 32) + qd32) * 1024);
      }
    }
  };

  // running state per tile: scores of query row c sit in lanes {c, c+16, c+32, c+48}, and so do the
  // statistics and (as O^T) the outputs of that row
  float m_run[T], l_run[T];
  f32x4 oacc[T][HT];
  int pos_q[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    m_run[t] = -INFINITY;
    l_run[t] = 0.f;
#pragma unroll
    for (int j = 0; j < HT; ++j) oacc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int rr = (qt0 + t) * 16 + c;
    pos_q[t] = cl.start_pos + (rr < R ? rr - div_small(rr, m_rinv) * m : 0);
  }

  // T = 1: keys and values of a step are both requested a step ahead, into registers.  T = 2: the
  // keys are; the values come through the wave's LDS buffer.  This wave's vector-memory operations
  // complete in the order issued, and the order is: keys 0, values 0, keys 1 (all landed before
  // step 0) | step 0: values 1, keys 2 | step 1: values 2, keys 3 | ..  So a step's values have
  // landed once at most the loads of the next step's keys (if there is a next step) are outstanding.
  constexpr bool V_AHEAD = T == 1;
  auto consume = [&](const KRegs& bk, VRegs& bv, int it) {
    const int tok0 = span0 + it * kStreamWgTokens + w * 32;
    if (tok0 >= total) return;  // (wave-uniform) nothing cached there
    asm volatile("" ::: "memory");  // the queries are read from LDS in every step, not kept in registers
    // all 32 tokens are cached tokens that every row of the pass sees: no masks needed
    const bool full = tok0 + 31 <= cl.start_pos;
    bf16x8 kf[2][KSQ], vf[HT];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int s = 0; s < KSQ; ++s) kf[tt][s] = __builtin_bit_cast(bf16x8, bk.k[tt][s]);
    if constexpr (V_AHEAD) {
#pragma unroll
      for (int j = 0; j < HT; ++j) vf[j] = __builtin_bit_cast(bf16x8, au32x4{bv.lo[j].x, bv.lo[j].y, bv.hi[j].x, bv.hi[j].y});
    } else {
      if (it + 1 < nsteps)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * KSQ) : "memory");
      else
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
      for (int j = 0; j < HT; ++j) {
        const au32x2 lo = *(const au32x2*)(vbuf + (j * 16 + c) * (kBlockTokens * 2) + g * 8);
        const au32x2 hi = *(const au32x2*)(vbuf + HD * kBlockTokens * 2 + (j * 16 + c) * (kBlockTokens * 2) + g * 8);
        vf[j] = __builtin_bit_cast(bf16x8, au32x4{lo.x, lo.y, hi.x, hi.y});
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the buffer has been read: it can take the next step's values
    }
    if (!full) {
      // values of tokens at or beyond `total` read as zero (their weights are exact zeros, but what the
      // cache holds there need not be a number); their keys need nothing: those scores are masked below
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        const int nvalid = min(4, max(0, total - (tok0 + tt * 16 + g * 4)));
        const unsigned long long keep = nvalid >= 4 ? ~0ull : ((1ull << (16 * nvalid)) - 1ull);
        const unsigned k0 = (unsigned)keep, k1 = (unsigned)(keep >> 32);
#pragma unroll
        for (int j = 0; j < HT; ++j) {
          au32x4 v = __builtin_bit_cast(au32x4, vf[j]);
          if (tt == 0) { v.x &= k0; v.y &= k1; } else { v.z &= k0; v.w &= k1; }
          vf[j] = __builtin_bit_cast(bf16x8, v);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (qt0 + t >= nqt) break;  // (workgroup-uniform)
      float sc[8];
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KSQ; ++s) {
          const bf16x8 qhi = __builtin_bit_cast(bf16x8, q_lds[((t * KSQ + s) * 2 + 0) * 64 + lane]);
          const bf16x8 qlo = __builtin_bit_cast(bf16x8, q_lds[((t * KSQ + s) * 2 + 1) * 64 + lane]);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[tt][s], qhi, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[tt][s], qlo, acc, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) sc[tt * 4 + i] = acc[i] * scale;
      }
      if constexpr (!V_AHEAD) {
        // The next step's values are asked for here, behind the first tile's scores: every key
        // fragment of the step has been used by now, so the compiler's waits for them, which do not
        // count these copies, have all been passed and none of them ends up waiting for the copies.
        // (Asked for without a branch, which would put a block boundary between the multiplies and
        // the first use of their results: the last step asks for its own values again, never read.)
        if (t == 0) {
          __builtin_amdgcn_sched_barrier(0);
          request_v_lds(min(it + 1, nsteps - 1));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (!full) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (tok0 + (i >> 2) * 16 + g * 4 + (i & 3) > pos_q[t]) sc[i] = -INFINITY;
      }
      float m_new = sc[0];
#pragma unroll
      for (int i = 1; i < 8; ++i) m_new = fmaxf(m_new, sc[i]);
      m_new = fold_groups(m_new, LaneMax{});
      m_new = fmaxf(m_new, m_run[t]);
      const float m_ref = (m_new == -INFINITY) ? 0.f : m_new;  // a row that has seen no token yet: all weights 0
      const float alpha = attn_exp(m_run[t] - m_ref);          // e^-inf = 0 for the first tokens a row sees
      float pv[8], l_step = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        pv[i] = attn_exp(sc[i] - m_ref);
        l_step += pv[i];
      }
      l_step = fold_groups(l_step, LaneAdd{});
      l_run[t] = l_run[t] * alpha + l_step;
      m_run[t] = m_new;
      bf16x8 phi, plo;
      split_hi_lo8(pv, phi, plo);
#pragma unroll
      for (int j = 0; j < HT; ++j) {
        f32x4 acc = oacc[t][j] * alpha;
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[j], phi, acc, 0, 0, 0);
        oacc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[j], plo, acc, 0, 0, 0);
      }
    }
  };

  KRegs ka, kb;
  VRegs va, vb;
  request_k(ka, 0);
  if constexpr (V_AHEAD) request_v(va, 0); else request_v_lds(0);
  if (nsteps > 1) {
    request_k(kb, 1);
    if constexpr (V_AHEAD) request_v(vb, 1);
  }
#pragma unroll
  for (int i = 0; i < QPT; ++i) {
    const int piece = tid + i * kStreamWaves * 64;
    const int hl = piece / (16 * (HD / 8)), rem = piece % (16 * (HD / 8)), qc = rem / (HD / 8), j = rem % (HD / 8);
    if (piece < QCH) {
#pragma unroll
      for (int t = 0; t < T; ++t) q_lds[((t * KSQ + (j >> 2)) * 2 + hl) * 64 + (j & 3) * 16 + qc] = qreg[t][i];
    }
  }
  __syncthreads();
  for (int it = 0; it < nsteps; it += 2) {
    consume(ka, va, it);
    if (it + 2 < nsteps) {
      request_k(ka, it + 2);
      if constexpr (V_AHEAD) request_v(va, it + 2);
    }
    if (it + 1 < nsteps) {
      consume(kb, V_AHEAD ? vb : va, it + 1);
      if (it + 3 < nsteps) {
        request_k(kb, it + 3);
        if constexpr (V_AHEAD) request_v(vb, it + 3);
      }
    }
  }

  // (T = 2: a wave that found nothing cached in its last steps never waited for the values it had
  // requested; they must have landed before its merge rows, the same LDS, are written)
  if constexpr (!V_AHEAD) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  // (The last products may have been issued in another basic block, where the compiler pads too few
  // wait states for the LDS stores of their results below: spell them out.)
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  // ---- merge of the waves, tile after tile: thread -> (query row, 8 consecutive elements) ----
  constexpr int TPR = HD / 8;
  const int mr = tid / TPR, e0 = (tid % TPR) * 8;
  float* gpart = part + cl.part_off + (size_t)(kvh * nz + zt) * cl.nsplit * (T * 16 * ROW);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    if (qt0 + t >= nqt) break;
    if (t > 0) __syncthreads();  // the merge of the tile before has read the LDS this tile writes
#pragma unroll
    for (int j = 0; j < HT; ++j) *(f32x4*)&o_lds[w][c][j * 16 + g * 4] = oacc[t][j];  // O[query c][element j*16 + g*4 + i]
    if (g == 0) {
      m_lds[w][c] = m_run[t];
      l_lds[w][c] = l_run[t];
    }
    __syncthreads();
    if (mr < 16) {
      float M = m_lds[0][mr];
#pragma unroll
      for (int ww = 1; ww < kStreamWaves; ++ww) M = fmaxf(M, m_lds[ww][mr]);
      const float M_ref = (M == -INFINITY) ? 0.f : M;
      float L = 0.f;
      f32x4 oa = f32x4{0.f, 0.f, 0.f, 0.f}, ob = oa;
#pragma unroll
      for (int ww = 0; ww < kStreamWaves; ++ww) {
        const float sw = attn_exp(m_lds[ww][mr] - M_ref);
        L += l_lds[ww][mr] * sw;
        oa += *(const f32x4*)&o_lds[ww][mr][e0] * sw;
        ob += *(const f32x4*)&o_lds[ww][mr][e0 + 4] * sw;
      }
      const int rr2 = (qt0 + t) * 16 + mr;
      if (rr2 < R) {
        if (cl.nsplit == 1) {
          const int g2 = div_small(rr2, m_rinv);
          const int head2 = kvh * group + g2, r2 = rr2 - g2 * m;
          const float y8[8] = {oa[0] / L, oa[1] / L, oa[2] / L, oa[3] / L, ob[0] / L, ob[1] / L, ob[2] / L, ob[3] / L};
          store_act8x<false>((u32x4*)outp, cl.row_off + r2, head2 * HD + e0, y8, act_tiles);
        } else {
          float* dst = gpart + ((size_t)(split * T + t) * 16 + mr) * ROW;
          Xwg<true>::st4f(dst + e0, oa);
          Xwg<true>::st4f(dst + e0 + 4, ob);
          if (e0 == 0) Xwg<true>::st4f(dst + HD, f32x4{M, L, 0.f, 0.f});
        }
      }
    }
  }
  if (cl.nsplit == 1) return;

  // ---- count in; the last of the client's splits to arrive merges them ----
  Xwg<true>::drain();  // this thread's partial stores have been acknowledged
  __syncthreads();
  unsigned* counter = counters + cl.count_off + kvh * nz + zt;
  if (tid == 0) {
    const unsigned prev = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int last = prev == (unsigned)cl.nsplit - 1u;
    if (last) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
    *last_lds = last;
  }
  __syncthreads();
  if (*last_lds == 0) return;
  for (int t = 0; t < T; ++t) {
    const int rr2 = (qt0 + t) * 16 + mr;
    if (qt0 + t >= nqt || mr >= 16 || rr2 >= R) continue;
    const int g2 = div_small(rr2, m_rinv);
    const int head2 = kvh * group + g2, r2 = rr2 - g2 * m;
    float acc[8];
    attn_merge_rows([&](int sp) { return gpart + ((size_t)(sp * T + t) * 16 + mr) * ROW; }, cl.nsplit, HD, e0, acc);
    store_act8x<false>((u32x4*)outp, cl.row_off + r2, head2 * HD + e0, acc, act_tiles);
  }
}

// ------------------------------------------------------------------------------------------------
// bf16 cache, passes of many prompt rows
// ------------------------------------------------------------------------------------------------
// The streaming kernel's results, bit for bit, with keys and values shared by four query tiles: workgroup (kv head,
// four query tiles, share of a block's spans) of four waves, a query tile each.  All waves walk the same tokens,
// 32 per step: a step's keys and values are copied from memory into LDS once for all tiles, two steps
// ahead, into a ring of three steps, one barrier per step.  What the streaming kernel gives its wave w (tokens
// it*128 + w*32 .. + 31 of every step of a span) is here every fourth step, so a wave keeps four running
// (max, sum, O), one per wave of the streaming kernel, merges them in the same order at the end of a span and leaves the
// span's partial in the scratch.  A workgroup that has all spans of its block merges them by itself, every wave its own;
// if several share them, partials are written through and the last to arrive merges, as in the streaming kernel.
//
// Every product, sum and rounding is the streaming kernel's own, in its order (the order of tokens inside an operand
// too); products with weights that are all zero and rescaling of zeros or by 1 are left out, which changes no bit of a
// finite result.  So which of the two kernels a pass takes, and into how many shares it is cut, is a matter of time alone
// (attn_prompt_shares): a row's result depends on its block's rows and context only.
//
// 8B shape, per layer, streaming / this kernel: 2047 rows 241 / 113 to 117 us, 333 rows behind 1000 tokens 69 / 39.  Bound by what a step
// waits for, with few waves to cover it: four states take 254 registers, so two waves share a SIMD (1.6 on average),
// each going from scores over a maximum, exponentials and cuts to 16 bits to the values' products.  Of
// the cycles the vector units issue in 47 %, the matrix cores work in 26 %, LDS is read in 33 %, 39 % of those bank conflicts: a
// lane needs 8 bytes of either block's values, and 16 lanes of such reads meet half of the banks.  Sums grouped otherwise
// (one state per wave, spans of 2048 tokens, a step's tokens in another order: three waves per SIMD) took 81 us for the 2047
// rows, but moved cached keys and values by a bf16 step here and there, and with them drawn tokens.
constexpr int kPromptRing = 3;  // steps in LDS
template <int HD>
constexpr size_t prompt_lds_bytes() { return (size_t)kPromptRing * (HD / 8) * 1024 + 16; }

// (grid: kv heads, groups of four tiles of the largest block, shares of all blocks; the last blocks have the longest
// contexts: their workgroups start first)
template <int HD>
__global__ __launch_bounds__(kStreamWaves * 64, 2) void attn_prompt_kernel(const float* q, KvView kv, int layer, int n_q_heads,
                                                                           AttnBatch batch, PromptShares shares, float* part,
                                                                           uint4* outp, int act_tiles, unsigned* counters) {
// (a product and a sum make one operation exactly where they do in the streaming kernel: spelled out)
#pragma clang fp contract(off)
  extern __shared__ float lds[];
  constexpr int KSQ = HD / 32, HT = HD / 16, ROW = HD + 4;
  constexpr int NI = HD / 8, NPW = NI / kStreamWaves;  // 1 KB copies of a step (keys, then values), per wave
  constexpr int kBuf = NI * 1024, kRing = kPromptRing * kBuf;
  const int kvh = blockIdx.x;
  int ci = 0, share = (int)(gridDim.z - 1 - blockIdx.z);
  while (share >= shares.n[ci]) share -= shares.n[ci++];
  const AttnClient cl = batch.c[ci];
  const int n_shares = shares.n[ci];
  const int group = n_q_heads / kv.n_kv_heads, m = cl.m, R = group * m;
  const int nqt = (R + 15) / 16, qt0 = (int)blockIdx.y * kStreamWaves;
  if (qt0 >= nqt) return;  // whole workgroup
  char* ring = (char*)lds;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int total = cl.start_pos + m;
  // this workgroup's spans, and the steps (of the whole context) they end with
  const int sp0 = share * cl.nsplit / n_shares, sp1 = (share + 1) * cl.nsplit / n_shares, span_steps = cl.span / kPromptStep;
  const int nsteps = min((total + kPromptStep - 1) / kPromptStep, sp1 * span_steps);
  const uint16_t* pool = (const uint16_t*)kv.pool;
  const int32_t* table = kv.table + cl.table_off;
  const float scale = 1.0f / sqrtf((float)HD);
  const float m_rinv = __builtin_amdgcn_rcpf((float)m);
  const int qd = n_q_heads * HD;

  // ---- copies: in memory's order but for a swap of 16-byte pieces inside a token's keys (a pair of value halves), so
  // that the reads of keys meet no bank twice (those of values, 8 bytes a lane, meet half of them).  Wave w copies half w % 2 of block w / 2 of a step; lane L
  // holds that block's table entry of step 64 n + L. ----
  constexpr int PIECES = HD / 8, TPC = 64 / PIECES;  // 16-byte pieces of a token's keys, tokens of a copy
  auto key_swap = [](int tok) { return PIECES == 16 ? tok : (tok >> 1) & (PIECES - 1); };
  const int blk_w = w >> 1, half_w = w & 1;
  int step_blk = 0;
  auto look_up = [&](int it) {
    const int tb = (it + lane) * kPromptStep + blk_w * kBlockTokens;
    step_blk = table[tb < total ? tb / kBlockTokens : 0];
  };
  int it = sp0 * span_steps;
  look_up(it & ~63);

  // ---- this wave's tile: rows, queries (hi and lo operands), first and last position ----
  const int tile = qt0 + w, rr0 = tile * 16, rr1 = min(rr0 + 15, R - 1);
  int pos_min = cl.start_pos, pos_max = -1;  // (no such tile: no token to see)
  if (tile < nqt) {
    const int h0 = div_small(rr0, m_rinv), h1 = div_small(rr1, m_rinv);
    pos_min = cl.start_pos + (h0 == h1 ? rr0 - h0 * m : 0);
    pos_max = cl.start_pos + (h0 == h1 ? rr1 - h1 * m : m - 1);
  }
  const int rr = rr0 + c;  // rows beyond the head group read row 0 of the group (their results are dropped)
  const bool live = rr < R;
  const int gq = live ? div_small(rr, m_rinv) : 0, r = live ? rr - gq * m : 0;
  const int pos_q = cl.start_pos + r;
  au32x4 qr[KSQ][2];
  {
    const uint16_t* q16 = (const uint16_t*)q + (size_t)(cl.row_off + r) * 2 * qd + (kvh * group + gq) * HD + g * 8;
#pragma unroll
    for (int s = 0; s < KSQ; ++s)
#pragma unroll
      for (int hl = 0; hl < 2; ++hl) qr[s][hl] = *(const au32x4*)(q16 + hl * qd + s * 32);
  }

  unsigned koff[NPW / 2];
#pragma unroll
  for (int i = 0; i < NPW / 2; ++i) {
    const int tok = (half_w * (NPW / 2) + i) * TPC + lane / PIECES;
    koff[i] = (unsigned)(tok * HD * 2 + ((lane % PIECES) ^ key_swap(tok)) * 16);
  }
  const unsigned voff = (unsigned)((lane >> 1) * 32 + ((lane & 1) ^ ((lane >> 4) & 1) ^ (lane >> 5)) * 16);
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)ring;
  auto request = [&](int it, int buf) {
    const char* base = (const char*)(pool + (int64_t)layer * kv.layer_stride +
                                     (int64_t)__builtin_amdgcn_readlane(step_blk, it & 63) * kv.block_elems + (int64_t)kvh * kBlockTokens * HD);
    const char* vbase = base + kv.v_offset * 2 + half_w * (NPW / 2) * 1024;
    const unsigned dst = lds0 + (unsigned)buf;
#pragma unroll
    for (int i = 0; i < NPW / 2; ++i) {
      lds_dma16(base, koff[i], dst + (blk_w * KSQ + half_w * (NPW / 2) + i) * 1024);
      lds_dma16(vbase + i * 1024, voff, dst + (2 * KSQ + (half_w * (NPW / 2) + i) * 2 + blk_w) * 1024);
    }
  };
  asm volatile("" : "+v"(step_blk));  // (awaited here; the queries are still on their way)
  request(it, 0);
  request(min(it + 1, nsteps - 1), kBuf);
  // (the queries: a wait for them inside the loop would be one for the copies, in every step)
  bf16x8 qf[KSQ][2];
#pragma unroll
  for (int s = 0; s < KSQ; ++s)
#pragma unroll
    for (int hl = 0; hl < 2; ++hl) {
      asm volatile("" : "+v"(qr[s][hl]));
      qf[s][hl] = __builtin_bit_cast(bf16x8, qr[s][hl]);
    }

  // operands from LDS: byte offsets in a step's buffer
  const int kat = c * HD * 2 + (g ^ key_swap(c)) * 16;  // (pieces 4 s + g of a token: the same with bits flipped)
  // (values: kilobytes of 32 elements' rows, of one block and of the other; element row e has its halves swapped if bits 3
  // and 4 of e differ.  Both blocks' parts of an operand are read by one instruction: rows e and e + 16 swapped alike
  // would have the compiler pair those instead, and copy registers behind.)
  const int vat = 2 * KSQ * 1024 + c * kBlockTokens * 2 + (g & 1) * 8;
  const int vat0 = vat + ((g >> 1) ^ (c >> 3)) * 16, vat1 = vat + 512 + ((g >> 1) ^ (c >> 3) ^ 1) * 16;
  auto key = [&](int b, int tt, int s) { return *(const bf16x8*)(ring + ((b + kat) ^ (s * 64)) + tt * KSQ * 1024); };
  auto value = [&](int b, int j) {
    const char* p = ring + (b + ((j & 1) ? vat1 : vat0)) + (j >> 1) * 2048;
    const au32x2 lo = *(const au32x2*)p, hi = *(const au32x2*)(p + 1024);
    return au32x4{lo.x, lo.y, hi.x, hi.y};
  };

  // the running state of query row c over the tokens of one wave of the streaming kernel
  struct State {
    f32x4 o[HT];
    float m, l;
  };
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  State st[kStreamWaves];

  // One step.  (The order is spelled out: left to itself the compiler reads the operands one by one, each right
  // before its products.)  edge: not every row sees all 32 tokens, or some are beyond the cached ones.  The lanes of a
  // row agree on a new maximum, and rescale, only in steps that bring one.  first: the state is still empty.
  auto step = [&](State& x, int b, int tok0, bool first, auto edge, auto request_next) {
    constexpr bool EDGE = decltype(edge)::value;
    bf16x8 kf[2][KSQ];
    au32x4 vr[HT];
#pragma unroll
    for (int s = 0; s < KSQ; ++s)
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) kf[tt][s] = key(b, tt, s);
    __builtin_amdgcn_sched_barrier(0);
    request_next();
    __builtin_amdgcn_sched_barrier(0);
    f32x4 sa[2];
#pragma unroll
    for (int s = 0; s < KSQ; ++s) {
#pragma unroll
      for (int hl = 0; hl < 2; ++hl)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
          sa[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[tt][s], qf[s][hl], s == 0 && hl == 0 ? zero : sa[tt], 0, 0, 0);
      if (!EDGE && s == KSQ / 2 - 1) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < HT; ++j) vr[j] = value(b, j);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    float sc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      sc[i] = sa[i >> 2][i & 3] * scale;
      if constexpr (EDGE) sc[i] = tok0 + (i >> 2) * 16 + g * 4 + (i & 3) > pos_q ? -INFINITY : sc[i];
    }
    float mx = sc[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) mx = fmaxf(mx, sc[i]);
    float alpha = 1.0f;
    if (__builtin_amdgcn_ballot_w64(mx > x.m) != 0) {
      const float m_new = fmaxf(fold_groups(mx, LaneMax{}), x.m);
      alpha = attn_exp(x.m - (m_new == -INFINITY ? 0.f : m_new));  // (0 for the first tokens a row sees)
      x.m = m_new;
      if (!first) {  // (uniform)
#pragma unroll
        for (int j = 0; j < HT; ++j) x.o[j] *= alpha;
      }
    }
    const float m_ref = x.m == -INFINITY ? 0.f : x.m;  // a row that has seen no token yet: all weights 0
    float pv[8], l_step = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      pv[i] = attn_exp(sc[i] - m_ref);
      l_step += pv[i];
    }
    l_step = fold_groups(l_step, LaneAdd{});
    x.l = __builtin_fmaf(x.l, alpha, l_step);
    bf16x8 phi, plo;
    split_hi_lo8(pv, phi, plo);
    if constexpr (EDGE) {
#pragma unroll
      for (int j = 0; j < HT; ++j) vr[j] = value(b, j);  // (read no earlier: registers)
      // values of tokens at or beyond `total` read as zero (their weights are exact zeros, but what the cache
      // holds there need not be a number)
      unsigned keep[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int nvalid = total - (tok0 + (i >> 1) * 16 + g * 4 + (i & 1) * 2);
        keep[i] = (nvalid > 0 ? 0xffffu : 0u) | (nvalid > 1 ? 0xffff0000u : 0u);
      }
#pragma unroll
      for (int j = 0; j < HT; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) vr[j][i] &= keep[i];
    }
#pragma unroll
    for (int j = 0; j < HT; ++j) x.o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vr[j]), phi, x.o[j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < HT; ++j) x.o[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vr[j]), plo, x.o[j], 0, 0, 0);
  };

  const int nfull = tile < nqt ? (pos_min + 1) / kPromptStep : 0;  // steps the tile sees in full
  const int nseen = tile < nqt ? pos_max / kPromptStep + 1 : 0;    // steps it sees anything of
  int rd = 0;
  auto open_step = [&] {
    // the step has landed for every wave, and every wave has read the step before: its buffer takes the step after the next
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(NPW) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto request_next = [&] {
    const int nx = min(it + 2, nsteps - 1);
    if ((nx & 63) == 0) {
      look_up(nx);
      asm volatile("" : "+v"(step_blk));  // (awaited here: at the join the compiler would wait in every step, for the copies as well)
    }
    request(nx, rd == 0 ? 2 * kBuf : rd - kBuf);
    rd = rd == kRing - kBuf ? 0 : rd + kBuf;
  };
  // the tile's partials: [span][element j*16 + g*4 .. + 3][lane], whole kilobytes, then (max, sum) of its 16 rows
  f32x4* tpart = (f32x4*)(part + cl.part_off + (size_t)(kvh * nqt + tile) * cl.nsplit * (16 * ROW));
  // (a workgroup that has all spans keeps the last one's)
  const int sp_kept = n_shares == 1 ? cl.nsplit - 1 : -1;
  f32x4 o[HT];
  float L = 0.f, M = 0.f;
#pragma unroll 1
  for (int sp = sp0; sp < sp1; ++sp) {
#pragma unroll
    for (int ww = 0; ww < kStreamWaves; ++ww) {
      st[ww].m = -INFINITY;
      st[ww].l = 0.f;
#pragma unroll
      for (int j = 0; j < HT; ++j) st[ww].o[j] = zero;
    }
    const int begin = it, end = min(nsteps, (sp + 1) * span_steps);
#pragma unroll 1
    while (it + kStreamWaves <= min(end, nfull)) {
#pragma unroll
      for (int ww = 0; ww < kStreamWaves; ++ww) {
        open_step();
        step(st[ww], rd, 0, it < begin + kStreamWaves, std::false_type{}, request_next);
        ++it;
      }
    }
#pragma unroll 1
    while (it < end) {
#pragma unroll
      for (int ww = 0; ww < kStreamWaves; ++ww) {
        if (it >= end) break;
        open_step();
        if (it < nseen) step(st[ww], rd, it * kPromptStep, it < begin + kStreamWaves, std::true_type{}, request_next);
        else request_next();  // (other waves' tiles see more)
        ++it;
      }
    }
    // (The last products may have been issued in another basic block, where the compiler pads too few
    // wait states for the reads of their results below: spell them out.)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    M = st[0].m;
#pragma unroll
    for (int ww = 1; ww < kStreamWaves; ++ww) M = fmaxf(M, st[ww].m);
    const float M_ref = M == -INFINITY ? 0.f : M;
    L = 0.f;
#pragma unroll
    for (int j = 0; j < HT; ++j) o[j] = zero;
#pragma unroll
    for (int ww = 0; ww < kStreamWaves; ++ww) {
      const float sw = attn_exp(st[ww].m - M_ref);
      L = __builtin_fmaf(st[ww].l, sw, L);
#pragma unroll
      for (int j = 0; j < HT; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[j][i] = __builtin_fmaf(st[ww].o[j][i], sw, o[j][i]);
    }
    if (sp != sp_kept && tile < nqt) {
      f32x4* dst = tpart + sp * (4 * ROW);
      const f32x4 ml = f32x4{M, L, 0.f, 0.f};  // (the four lanes of a row write the same)
      if (n_shares > 1) {  // written through to memory: another workgroup may merge
#pragma unroll
        for (int j = 0; j < HT; ++j) Xwg<true>::st4f((float*)(dst + j * 64 + lane), o[j]);
        Xwg<true>::st4f((float*)(dst + HT * 64 + c), ml);
      } else {
#pragma unroll
        for (int j = 0; j < HT; ++j) dst[j * 64 + lane] = o[j];
        dst[HT * 64 + c] = ml;
      }
    }
  }
  // copies asked for past the end land before the LDS is given back; this thread's partial stores have been acknowledged
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (n_shares > 1) {  // count in; the last of the block's workgroups to arrive merges
    __syncthreads();
    int* last_lds = (int*)(ring + kRing);
    if (tid == 0) {
      unsigned* counter = counters + cl.count_off + kvh * (int)gridDim.y + (int)blockIdx.y;
      const unsigned prev = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int last = prev == (unsigned)n_shares - 1u;
      if (last) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
      *last_lds = last;
    }
    __syncthreads();
    if (*last_lds == 0) return;
  }
  if (tile >= nqt) return;

  // ---- the spans' partials, as attn_merge_rows takes them ----
  if (cl.nsplit > 1) {
    constexpr int BATCH = 9;
    auto max_of = [&](int s) { return s == sp_kept ? M : tpart[s * (4 * ROW) + HT * 64 + c][0]; };
    float top = -INFINITY, sum = 0.f;
    f32x4 acc[HT];
#pragma unroll
    for (int j = 0; j < HT; ++j) acc[j] = zero;
    for (int s0 = 0; s0 < cl.nsplit; s0 += BATCH) {
      const int s1 = min(cl.nsplit, s0 + BATCH);
      float bm = top;
      for (int s = s0; s < s1; ++s) bm = fmaxf(bm, max_of(s));
      const float so = top == -INFINITY ? 0.f : attn_exp(top - bm);
      for (int s = s0; s < s1; ++s) {
        const f32x4* ps = tpart + s * (4 * ROW);
        f32x4 os[HT];
        float m_s = M, l_s = L;
        if (s == sp_kept) {
#pragma unroll
          for (int j = 0; j < HT; ++j) os[j] = o[j];
        } else {
          const f32x4 ml = ps[HT * 64 + c];
          m_s = ml[0];
          l_s = ml[1];
#pragma unroll
          for (int j = 0; j < HT; ++j) os[j] = ps[j * 64 + lane];
        }
        const float wgt = m_s != -INFINITY ? attn_exp(m_s - bm) : 0.f;
        // (the first of a batch: the product is rounded, the rescaling is part of the sum)
        auto take = [&](float a, float v) { return s == s0 ? __builtin_fmaf(a, so, v * wgt) : __builtin_fmaf(v, wgt, a); };
        sum = take(sum, l_s);
#pragma unroll
        for (int j = 0; j < HT; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[j][i] = take(acc[j][i], os[j][i]);
      }
      top = bm;
    }
    L = sum;
#pragma unroll
    for (int j = 0; j < HT; ++j) o[j] = acc[j];
  }
#pragma unroll
  for (int j = 0; j < HT; ++j) {
    const f32x4 y = f32x4{o[j][0] / L, o[j][1] / L, o[j][2] / L, o[j][3] / L}, y2 = from16(y);  // (elements + 4 .. + 7 of the 8)
    const float y8[8] = {y[0], y[1], y[2], y[3], y2[0], y2[1], y2[2], y2[3]};
    if (live && (g & 1) == 0) store_act8x<false>((u32x4*)outp, cl.row_off + r, (kvh * group + gq) * HD + j * 16 + g * 4, y8, act_tiles);
  }
}

// grid = (threads of the largest client / 64, clients)
__global__ __launch_bounds__(64) void attn_merge_packed_kernel(const float* part, int n_q_heads, int h, AttnBatch batch,
                                                              uint4* outp, int act_tiles, const int32_t* gate) {
  if (gate != nullptr && *gate == 0) return;
  const AttnClient c = batch.c[blockIdx.y];
  attn_merge_thread<false>(part + c.part_off, c.m, n_q_heads, h, c.nsplit, (u32x4*)outp,
                           blockIdx.x * blockDim.x + threadIdx.x, c.row_off, act_tiles);
}

// merge the splits of one (row, head): o = sum_s e^{m_s - M} o_s / sum_s e^{m_s - M} l_s, splits taken
// in index order.  ceil(h/8) threads per (row, head), 8 consecutive elements each (fp32 cache path).
__global__ __launch_bounds__(256) void attn_combine_kernel(const float* __restrict__ part, int m, int n_q_heads, int h,
                                                           int nsplit, float* __restrict__ out) {
  const int tpp = (h + 7) / 8;  // threads per pair
  const int gt = blockIdx.x * blockDim.x + threadIdx.x;
  const int pair = gt / tpp, e0 = (gt % tpp) * 8;  // pair = head * m + r
  if (pair >= m * n_q_heads) return;
  const int head = pair / m, r = pair % m;
  const float* p = part + (size_t)pair * nsplit * (h + kPartPad);
  float M = -INFINITY;
  for (int s = 0; s < nsplit; ++s) M = fmaxf(M, p[(size_t)s * (h + kPartPad) + h]);
  float L = 0.f, acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  for (int s = 0; s < nsplit; ++s) {
    const float* ps = p + (size_t)s * (h + kPartPad);
    const float ms = ps[h];
    if (ms == -INFINITY) continue;
    const float wgt = expf(ms - M);
    L += ps[h + 1] * wgt;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] += ps[min(e0 + i, h - 1)] * wgt;
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] /= L;
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (e0 + i < h) out[((size_t)r * n_q_heads + head) * h + e0 + i] = acc[i];
}

int attn_nsplit(int total_tokens, int chunk) { return (total_tokens + chunk - 1) / chunk; }

hipError_t launch_attention(const AttnCall& c, hipStream_t st) {
  const int h = c.kv.head_dim;
  const int total = c.start_pos + c.m;
  const int nsplit = attn_nsplit(total, c.chunk);
  if (c.dtype == PIPESD_F32 && h % 16 == 0) {
    if (c.chunk != kAttnF32Split) return hipErrorInvalidValue;
    const hipError_t e = launch_attn_f32(c, nsplit, st);
    if (e != hipSuccess || nsplit == 1) return e;
  } else if (c.dtype == PIPESD_F32) {
    if (c.chunk > kAttnChunkMax || c.m > kMaxRows) return hipErrorInvalidValue;
    const size_t lds = (size_t)(2 * kAttnChunkMax * (h + 1) + kMaxRows * h + kMaxRows * kAttnChunkMax) * sizeof(float);
    dim3 grid(c.kv.n_kv_heads, nsplit);
    attn_partial_kernel<float><<<grid, kAttnThreads, lds, st>>>(c.q, c.kv, c.layer, c.m, c.start_pos, c.n_q_heads,
                                                                c.chunk, nsplit, c.part);
  } else {
    const AttnBatch& b = c.batch;
    if (b.n < 1 || b.n > kMaxPassClients) return hipErrorInvalidValue;
    const int group = c.n_q_heads / c.kv.n_kv_heads;
    int splits = 0, max_m = 1;
    long tasks = 0;  // (kv head, split, query tile) over all clients
    for (int i = 0; i < b.n; ++i) {
      splits += b.c[i].nsplit;
      max_m = b.c[i].m > max_m ? b.c[i].m : max_m;
      tasks += (long)c.kv.n_kv_heads * b.c[i].nsplit * ((group * b.c[i].m + 15) / 16);
    }
    if (c.stream_tiles) {  // few rows per client: the streaming kernel (the batch was planned by attn_stream_plan)
      const int T = c.stream_tiles;
      if ((h != 128 && h != 64) || max_m > kPromptBlockRows || (T != 1 && T != 2) || c.counters == nullptr) return hipErrorInvalidValue;
      for (int i = 0; i < b.n; ++i)  // (a lane per step holds the step's block-table entries)
        if (b.c[i].span < kStreamWgTokens || b.c[i].span > kStreamMaxSteps * kStreamWgTokens) return hipErrorInvalidValue;
      using std::integral_constant;
      PromptShares shares;
      if (const int n = attn_prompt_shares(group, c.kv.n_kv_heads, h, device_cu_count(), b, &shares)) {
        if (c.gate != nullptr) return hipErrorInvalidValue;
        const dim3 grid(c.kv.n_kv_heads, (attn_query_tiles(group, max_m) + kStreamWaves - 1) / kStreamWaves, n);
        auto go = [&](auto hd) -> hipError_t {
          constexpr int HD = decltype(hd)::value;
          static_assert(prompt_lds_bytes<HD>() <= 64 * 1024, "no limit to raise");
          attn_prompt_kernel<HD><<<grid, kStreamWaves * 64, prompt_lds_bytes<HD>(), st>>>(
              c.q, c.kv, c.layer, c.n_q_heads, b, shares, c.part, (uint4*)c.outp, c.act_tiles, c.counters);
          return hipGetLastError();
        };
        return h == 128 ? go(integral_constant<int, 128>{}) : go(integral_constant<int, 64>{});
      }
      AttnBatch ordered = b;
      const StreamItems items = attn_stream_items(group, T, ordered);
      const dim3 grid = b.n > 1 ? dim3(c.kv.n_kv_heads, items.n)
                                : dim3(c.kv.n_kv_heads, b.c[0].nsplit, (attn_query_tiles(group, b.c[0].m) + T - 1) / T);
      const dim3 block(kStreamWaves * 64);
      auto go = [&](auto hd, auto t) -> hipError_t {
        constexpr int HD = decltype(hd)::value, TT = decltype(t)::value;
        static std::atomic<uint64_t> lds_allowed;
        constexpr size_t lds = stream_lds_bytes<HD>(TT);
        const hipError_t e = allow_lds(lds_allowed, (const void*)attn_stream_kernel<HD, TT>, lds);
        if (e != hipSuccess) return e;
        attn_stream_kernel<HD, TT><<<grid, block, lds, st>>>(c.q, c.kv, c.layer, c.n_q_heads, ordered, items, c.part, (uint4*)c.outp,
                                                             c.act_tiles, c.gate, c.counters);
        return hipGetLastError();
      };
      if (h == 128) return T == 2 ? go(integral_constant<int, 128>{}, integral_constant<int, 2>{}) : go(integral_constant<int, 128>{}, integral_constant<int, 1>{});
      return T == 2 ? go(integral_constant<int, 64>{}, integral_constant<int, 2>{}) : go(integral_constant<int, 64>{}, integral_constant<int, 1>{});
    }
    // more tasks than the device holds at once (two workgroups per compute unit): a workgroup walks
    // several query tiles with its keys and values in registers, as many as still leave about two
    // workgroups per compute unit (a 128-row prompt block has 32 tiles per (kv head, split))
    const int max_qt = (group * max_m + 15) / 16, n_cu = device_cu_count();
    const int qpw = tasks > 4L * n_cu ? (int)std::max(1L, std::min((long)max_qt, tasks / (2L * n_cu))) : 1;
    dim3 grid(c.kv.n_kv_heads, splits, (max_qt + qpw - 1) / qpw);
    if (h != 128 && h != 64) return hipErrorInvalidValue;
    const size_t lds = attn_lds_floats(h) * sizeof(float);
    const dim3 block(kAttnWaves * 64);
    auto go = [&](auto hd, auto multi) -> hipError_t {
      constexpr int HD = decltype(hd)::value;
      constexpr bool MULTI = decltype(multi)::value;
      static std::atomic<uint64_t> lds_allowed;
      const hipError_t ea = allow_lds(lds_allowed, (const void*)attn_mfma_kernel<HD, MULTI>, lds);
      if (ea != hipSuccess) return ea;
      attn_mfma_kernel<HD, MULTI><<<grid, block, lds, st>>>(c.q, c.kv, c.layer, c.n_q_heads, b, c.part, qpw, c.gate);
      return hipSuccess;
    };
    using std::integral_constant;
    hipError_t el;
    if (h == 128) el = qpw > 1 ? go(integral_constant<int, 128>{}, std::true_type{}) : go(integral_constant<int, 128>{}, std::false_type{});
    else el = qpw > 1 ? go(integral_constant<int, 64>{}, std::true_type{}) : go(integral_constant<int, 64>{}, std::false_type{});
    if (el != hipSuccess) return el;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (c.dtype == PIPESD_F32) {
    const int threads = c.m * c.n_q_heads * ((h + 7) / 8);
    attn_combine_kernel<<<(threads + 255) / 256, 256, 0, st>>>(c.part, c.m, c.n_q_heads, h, nsplit, c.out);
  } else {
    int max_m = 1;
    for (int i = 0; i < c.batch.n; ++i) max_m = c.batch.c[i].m > max_m ? c.batch.c[i].m : max_m;
    const int threads = max_m * c.n_q_heads * (h / 8);
    attn_merge_packed_kernel<<<dim3((threads + 63) / 64, c.batch.n), 64, 0, st>>>(c.part, c.n_q_heads, h, c.batch,
                                                                                   (uint4*)c.outp, c.act_tiles, c.gate);
  }
  return hipGetLastError();
}

int attn_chunk_tokens(int dtype, int head_dim) {
  if (dtype != PIPESD_F32) return kAttnWgTokens;
  return head_dim % 16 == 0 ? kAttnF32Split : kAttnChunkMax;
}

}  // namespace pipesd
