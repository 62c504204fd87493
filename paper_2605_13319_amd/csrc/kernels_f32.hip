// The fp32 model's layer kernels, on the fp32 matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands,
// fp32 accumulation).  (The target forward of Sec. 2.1 / 2.2.)
//
// These models are small and their passes are chains of short launches, so a launch is bound by its
// own latencies: everything it needs is requested at once by many waves, and what used to be
// launches of their own (norm, rotary + cache append, SiLU * up) is done where the operands are read
// or the results stored.
#include <type_traits>

#include "common.h"
#include "lds_limit.h"

namespace pipesd {

// ------------------------------------------------------------------------------------------------
// out[m][N] = act[m][K] * W[N][K]^T, with the norm in front and the epilogue behind it
// ------------------------------------------------------------------------------------------------
// Workgroup (16 weight rows, RT * 16 activation rows) of eight waves: wave w takes the blocks w, w + 8,
// .. of 16 columns.  Weights are the A operand, activations the B operand; within a block the matrix
// instruction j of four takes columns 4 g + j of lane group g, for both operands, so a lane's share of
// a block is 16 contiguous bytes of its row.  kAheadF32 blocks are requested at once.  The eight
// sums are added through LDS in pairs.  The norm needs the rows' sums of squares: the waves see every
// column of every row, so they gather them from the operands they load anyway, and the product of
// x * gain is scaled by the row's rstd at the end.
//
// Bound by the latency of the requests, not by bandwidth (5.3 MB of weights in all for 2 layers of
// width 256).  Two layers of that width: a round of 5 rows at a context of 128 takes 99 us, 264 with one
// wave per output column on the vector units and the norm, rotary and SiLU steps in launches of their
// own; a prompt of 120 tokens 52 us (its last layer ends behind its keys and values), 2340 before (a
// launch of 32 rows: 84 us, now 7 for all 119).
constexpr int kF32Waves = 8;
constexpr int kAheadF32 = 4;

template <bool VEC>  // VEC: rows of both operands start on 16-byte boundaries and K is a multiple of 4
__device__ __forceinline__ f32x4 load_cols(const float* row, int k, int K) {
  if constexpr (VEC) {
    const f32x4 v = *(const f32x4*)(row + min(k, K - 4));
    return k < K ? v : f32x4{0.f, 0.f, 0.f, 0.f};
  } else {
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = row[min(k + i, K - 1)];
      v[i] = k + i < K ? x : 0.f;
    }
    return v;
  }
}

// row of the weight matrix that row i of tile t multiplies (rows past the end: any valid row)
template <int EPI>
__device__ __forceinline__ int f32_weight_row(const GemmF32Call& a, int t, int i) {
  if constexpr (EPI == EPI_SWIGLU) {  // 8 gate rows and the 8 matching up rows
    const int F = a.N / 2, j = min(t * 8 + (i & 7), F - 1);
    return i < 8 ? j : F + j;
  } else if constexpr (EPI == EPI_QKV) {  // rows i..i+7 of a head and their rotary partners (head_dim a multiple of 16)
    const int h = a.kv.head_dim, hpt = h / 16;
    return (t / hpt) * h + (t % hpt) * 8 + (i & 7) + (i < 8 ? 0 : h / 2);
  } else {
    return min(t * 16 + i, a.N - 1);
  }
}

template <int EPI, int RT, bool VEC>
__global__ __launch_bounds__(kF32Waves * 64) void gemm_f32_kernel(GemmF32Call a) {
  __shared__ f32x4 red[kF32Waves][RT][64];
  __shared__ float sqs[kF32Waves][RT][16];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int t = blockIdx.x, row0 = blockIdx.y * RT * 16;
  const bool norm = a.gain != nullptr;
  const float* wrow = a.w + (size_t)f32_weight_row<EPI>(a, t, c) * a.K;
  const float* xrow[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) xrow[rt] = a.act + (size_t)min(row0 + rt * 16 + c, a.m - 1) * a.lda;
  // eight sums per tile and row, by column of a lane's share and by parity of the block: short chains,
  // added in pairs (one chain per wave was 1.4 times as far off 64 bits)
  f32x4 acc[RT][8], sq[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[rt][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    sq[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // What the epilogue reads besides the sums is asked for with the first operands (wave rt finishes row tile rt; the
  // others read its rows again): behind the sums it would be one more round trip to memory.
  const int erow = min(row0 + min(w, RT - 1) * 16 + c, a.m - 1);
  f32x4 pre[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  int blk = 0;
  if constexpr (EPI == EPI_RESID) {
#pragma unroll
    for (int i = 0; i < 4; ++i) pre[0][i] = a.out[(size_t)erow * a.ldo + min(t * 16 + g * 4 + i, a.N - 1)];
  } else if constexpr (EPI == EPI_QKV) {
    const int h = a.kv.head_dim, hpt = h / 16;
    const float* cs = a.rope_cs + ((size_t)erow * (h / 2) + (t % hpt) * 8 + (g & 1) * 4) * 2;
#pragma unroll
    for (int i = 0; i < 8; ++i) pre[i >> 2][i & 3] = cs[i];
    blk = a.kv.table[(a.start_pos + erow) / kBlockTokens];
  }
  for (int k0 = w * 16; k0 < a.K; k0 += kF32Waves * 16 * kAheadF32) {
    f32x4 wf[kAheadF32], gf[kAheadF32], xf[RT][kAheadF32];
#pragma unroll
    for (int u = 0; u < kAheadF32; ++u) {
      const int k = k0 + u * kF32Waves * 16 + g * 4;  // (columns past K read as zero)
      wf[u] = load_cols<VEC>(wrow, k, a.K);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) xf[rt][u] = load_cols<VEC>(xrow[rt], k, a.K);
      gf[u] = norm ? load_cols<VEC>(a.gain, k, a.K) : f32x4{1.f, 1.f, 1.f, 1.f};
    }
#pragma unroll
    for (int u = 0; u < kAheadF32; ++u) {
      if (k0 + u * kF32Waves * 16 >= a.K) break;  // (uniform: nothing but zeros from here on)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const f32x4 x = xf[rt][u], y = x * gf[u];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          sq[rt][j] = fmaf(x[j], x[j], sq[rt][j]);
          f32x4& s = acc[rt][(u & 1) * 4 + j];
          s = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[u][j], y[j], s, 0, 0, 0);
        }
      }
    }
  }
  // (The last products may have been issued in another basic block, where the compiler pads no wait
  // states for the stores below: spell them out, once, behind all sums and in front of
  // whoever reads them.)
  auto tie = [&](int rt) {
    f32x4* s = acc[rt];
    asm volatile("" : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3]), "+v"(s[4]), "+v"(s[5]), "+v"(s[6]), "+v"(s[7]));
  };
#pragma unroll
  for (int rt = 1; rt < RT; ++rt) tie(rt);
  asm volatile("s_nop 15\n\ts_nop 7"
               : "+v"(acc[0][0]), "+v"(acc[0][1]), "+v"(acc[0][2]), "+v"(acc[0][3]), "+v"(acc[0][4]), "+v"(acc[0][5]),
                 "+v"(acc[0][6]), "+v"(acc[0][7]));
#pragma unroll
  for (int rt = 1; rt < RT; ++rt) tie(rt);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    red[w][rt][lane] = ((acc[rt][0] + acc[rt][1]) + (acc[rt][2] + acc[rt][3])) +
                       ((acc[rt][4] + acc[rt][5]) + (acc[rt][6] + acc[rt][7]));
    if (norm) {
      float q = (sq[rt][0] + sq[rt][1]) + (sq[rt][2] + sq[rt][3]);
      q = fold_groups(q, LaneAdd{});
      if (g == 0) sqs[w][rt][c] = q;
    }
  }
  __syncthreads();
  if (w >= RT) return;  // wave rt finishes row tile rt: lane (g, c) holds weight rows 4 g .. 4 g + 3 of row c
  const int row = row0 + w * 16 + c;
  static_assert(kF32Waves == 8, "the sums below");
  f32x4 v = ((red[0][w][lane] + red[1][w][lane]) + (red[2][w][lane] + red[3][w][lane])) +
            ((red[4][w][lane] + red[5][w][lane]) + (red[6][w][lane] + red[7][w][lane]));
  if (norm) {
    const float q = ((sqs[0][w][c] + sqs[1][w][c]) + (sqs[2][w][c] + sqs[3][w][c])) +
                    ((sqs[4][w][c] + sqs[5][w][c]) + (sqs[6][w][c] + sqs[7][w][c]));
    v = v * (1.0f / sqrtf(q / (float)a.K + a.eps));
  }
  const bool live = row < a.m;
  if constexpr (EPI == EPI_STORE || EPI == EPI_RESID) {
    float* o = a.out + (size_t)row * a.ldo + t * 16 + g * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (live && t * 16 + g * 4 + i < a.N) o[i] = EPI == EPI_RESID ? pre[0][i] + v[i] : v[i];
  } else if constexpr (EPI == EPI_SWIGLU) {
    f32x4 up;
#pragma unroll
    for (int i = 0; i < 4; ++i) up[i] = from32(v[i]);
    const int j0 = t * 8 + (g & 1) * 4, F = a.N / 2;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (live && g < 2 && j0 + i < F) a.out[(size_t)row * a.ldo + j0 + i] = (v[i] / (1.0f + expf(-v[i]))) * up[i];
  } else {
    f32x4 pt;
#pragma unroll
    for (int i = 0; i < 4; ++i) pt[i] = from32(v[i]);
    if (!live || g >= 2) return;
    const int h = a.kv.head_dim, half = h / 2, hpt = h / 16;
    const int hd = t / hpt, i0 = (t % hpt) * 8 + g * 4;
    f32x4 r0 = v, r1 = pt;
    if (hd < a.n_q_heads + a.kv.n_kv_heads) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float cs = pre[i >> 1][2 * (i & 1)], sn = pre[i >> 1][2 * (i & 1) + 1];
        r0[i] = v[i] * cs - pt[i] * sn;
        r1[i] = pt[i] * cs + v[i] * sn;
      }
    }
    float* kvp = (float*)a.kv.pool;
    const int pos = a.start_pos + row;
    if (hd < a.n_q_heads) {
      float* o = a.out + (size_t)row * a.ldo + hd * h + i0;
      *(f32x4*)o = r0;
      *(f32x4*)(o + half) = r1;
    } else if (hd < a.n_q_heads + a.kv.n_kv_heads) {
      float* o = kvp + k_index(a.kv, a.layer, blk, pos, hd - a.n_q_heads, i0);
      *(f32x4*)o = r0;
      *(f32x4*)(o + half) = r1;
    } else {
      float* o = kvp + v_index(a.kv, a.layer, blk, pos, hd - a.n_q_heads - a.kv.n_kv_heads, i0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        o[(size_t)i * kBlockTokens] = r0[i];
        o[(size_t)(half + i) * kBlockTokens] = r1[i];
      }
    }
  }
}

bool gemm_f32_fuses_rope(int head_dim) { return head_dim % 16 == 0; }

hipError_t launch_gemm_f32(const GemmF32Call& c, hipStream_t st) {
  if (c.m < 1 || c.N < 1 || c.K < 1 || (c.epi == EPI_QKV && !gemm_f32_fuses_rope(c.kv.head_dim)) ||
      (c.epi == EPI_SWIGLU && c.N % 2))
    return hipErrorInvalidValue;
  const bool vec = c.K % 4 == 0 && c.lda % 4 == 0;  // (the buffers themselves are the library's own, 256-byte aligned)
  const int tiles = c.epi == EPI_SWIGLU ? (c.N / 2 + 7) / 8 : (c.N + 15) / 16;
  // 16 rows per workgroup for the usual round, 32 beyond: half the reads of the weights, and still one
  // matrix-core chain per row tile
  const int rt = c.m <= 16 ? 1 : 2;
  const dim3 grid(tiles, (c.m + rt * 16 - 1) / (rt * 16)), block(kF32Waves * 64);
  auto launch = [&](auto epi) {
    constexpr int EPI = decltype(epi)::value;
    if (rt == 1 && vec) gemm_f32_kernel<EPI, 1, true><<<grid, block, 0, st>>>(c);
    else if (rt == 1) gemm_f32_kernel<EPI, 1, false><<<grid, block, 0, st>>>(c);
    else if (vec) gemm_f32_kernel<EPI, 2, true><<<grid, block, 0, st>>>(c);
    else gemm_f32_kernel<EPI, 2, false><<<grid, block, 0, st>>>(c);
  };
  switch (c.epi) {
    case EPI_STORE: launch(std::integral_constant<int, EPI_STORE>{}); break;
    case EPI_RESID: launch(std::integral_constant<int, EPI_RESID>{}); break;
    case EPI_SWIGLU: launch(std::integral_constant<int, EPI_SWIGLU>{}); break;
    case EPI_QKV: launch(std::integral_constant<int, EPI_QKV>{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// attention over the fp32 cache (head_dim a multiple of 16)
// ------------------------------------------------------------------------------------------------
// Workgroup (KV head, split of 256 tokens, 16 of the rows that share the KV head) of eight waves: wave
// w takes the cache blocks w and w + 8 of the split (16 tokens each), all of whose keys and values it
// requests at once.  S^T = K Q^T has the 16 tokens of a block in a lane's four registers and the four
// lane groups, for one query row per lane: exactly the B operand of O^T = V^T P, so the probabilities
// never leave their registers.  The waves' (max, sum, O) are merged through LDS in wave order; a
// context of one split is written normalised, otherwise the splits are merged by the combine kernel.
constexpr int kF32AttnSteps = 2;

template <int HT>
__global__ __launch_bounds__(kF32Waves * 64) void attn_f32_kernel(const float* __restrict__ q, KvView kv, int layer, int m,
                                                                  int start_pos, int n_q_heads, int nsplit,
                                                                  float* __restrict__ part, float* __restrict__ out) {
  constexpr int H = HT * 16, ROW = H + 4;
  extern __shared__ float lds[];
  float(*o_lds)[16][ROW] = (float(*)[16][ROW])lds;
  float(*m_lds)[16] = (float(*)[16])(lds + (size_t)kF32Waves * 16 * ROW);
  float(*l_lds)[16] = m_lds + kF32Waves;
  const int kvh = blockIdx.x, split = blockIdx.y, qt = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int group = n_q_heads / kv.n_kv_heads, R = group * m, total = start_pos + m;
  const int rr = qt * 16 + c;  // rows beyond the head group read its row 0 (their results are dropped)
  const int gq = rr < R ? rr / m : 0, r = rr < R ? rr - gq * m : 0;
  const int pos_q = start_pos + r;
  const float* pool = (const float*)kv.pool;
  const float scale = 1.0f / sqrtf((float)H);
  f32x4 qf[HT], kf[kF32AttnSteps][HT], vf[kF32AttnSteps][HT];
  int tok0[kF32AttnSteps];
#pragma unroll
  for (int s = 0; s < kF32AttnSteps; ++s) {
    tok0[s] = split * kAttnF32Split + (s * kF32Waves + w) * kBlockTokens;
    const int blk = kv.table[min(tok0[s], total - 1) / kBlockTokens];  // (a block past the context: any cached one, masked below)
    const float* base = pool + (int64_t)layer * kv.layer_stride + (int64_t)blk * kv.block_elems;
#pragma unroll
    for (int j = 0; j < HT; ++j) {
      kf[s][j] = *(const f32x4*)(base + ((int64_t)kvh * kBlockTokens + c) * H + j * 16 + g * 4);
      vf[s][j] = *(const f32x4*)(base + kv.v_offset + ((int64_t)kvh * H + j * 16 + c) * kBlockTokens + g * 4);
    }
  }
#pragma unroll
  for (int j = 0; j < HT; ++j) qf[j] = *(const f32x4*)(q + ((size_t)r * n_q_heads + kvh * group + gq) * H + j * 16 + g * 4);
  __builtin_amdgcn_sched_barrier(0);  // (all of it is asked for before the first use: left alone, the scheduler sinks the loads)

  f32x4 sc[kF32AttnSteps];
  float mx = -INFINITY;
#pragma unroll
  for (int s = 0; s < kF32AttnSteps; ++s) {
    f32x4 part4[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      part4[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < HT; ++j) part4[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[s][j][i], qf[j][i], part4[i], 0, 0, 0);
    }
    const f32x4 acc = (part4[0] + part4[1]) + (part4[2] + part4[3]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sc[s][i] = tok0[s] + g * 4 + i <= pos_q ? acc[i] * scale : -INFINITY;
      mx = fmaxf(mx, sc[s][i]);
    }
  }
  mx = fold_groups(mx, LaneMax{});
  const float ref = mx == -INFINITY ? 0.f : mx;  // (a row that sees none of this wave's tokens)
  float l = 0.f;
  f32x4 osum[kF32AttnSteps][HT];
#pragma unroll
  for (int s = 0; s < kF32AttnSteps; ++s) {
    f32x4 p;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[i] = expf(sc[s][i] - ref);
      l += p[i];
    }
#pragma unroll
    for (int j = 0; j < HT; ++j) {
      osum[s][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // values beyond the context read as zero (their weights are zeros, but the cache need not hold a number there)
        const float v = tok0[s] + g * 4 + i < total ? vf[s][j][i] : 0.f;
        osum[s][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, p[i], osum[s][j], 0, 0, 0);
      }
    }
  }
  l = fold_groups(l, LaneAdd{});
#pragma unroll
  for (int s = 0; s < kF32AttnSteps; ++s)
#pragma unroll
    for (int j = 0; j < HT; ++j) asm volatile("s_nop 15\n\ts_nop 7" : "+v"(osum[s][j]));
  static_assert(kF32AttnSteps == 2, "the sum below");
#pragma unroll
  for (int j = 0; j < HT; ++j) *(f32x4*)&o_lds[w][c][j * 16 + g * 4] = osum[0][j] + osum[1][j];
  if (g == 0) {
    m_lds[w][c] = mx;
    l_lds[w][c] = l;
  }
  __syncthreads();
  // thread -> (query row, 4 consecutive elements)
  const int mr = tid / (H / 4), e0 = (tid % (H / 4)) * 4, rr2 = qt * 16 + mr;
  if (mr >= 16 || rr2 >= R) return;
  float M = m_lds[0][mr];
#pragma unroll
  for (int ww = 1; ww < kF32Waves; ++ww) M = fmaxf(M, m_lds[ww][mr]);
  const float M_ref = M == -INFINITY ? 0.f : M;
  float L = 0.f;
  f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ww = 0; ww < kF32Waves; ++ww) {
    const float sw = expf(m_lds[ww][mr] - M_ref);
    L += l_lds[ww][mr] * sw;
    o += *(const f32x4*)&o_lds[ww][mr][e0] * sw;
  }
  const int head = kvh * group + rr2 / m, r2 = rr2 % m;
  if (nsplit == 1) {
    *(f32x4*)(out + ((size_t)r2 * n_q_heads + head) * H + e0) = o / L;
  } else {
    float* dst = part + (((size_t)head * m + r2) * nsplit + split) * ROW;
    *(f32x4*)(dst + e0) = o;
    if (e0 == 0) *(f32x4*)(dst + H) = f32x4{M, L, 0.f, 0.f};
  }
}

template <int HT>
static hipError_t launch_attn_f32_ht(const AttnCall& c, int nsplit, hipStream_t st) {
  constexpr size_t lds = ((size_t)kF32Waves * 16 * (HT * 16 + 4) + 2 * kF32Waves * 16) * sizeof(float);
  static std::atomic<uint64_t> lds_allowed;
  const hipError_t e = allow_lds(lds_allowed, (const void*)attn_f32_kernel<HT>, lds);
  if (e != hipSuccess) return e;
  const int group = c.n_q_heads / c.kv.n_kv_heads;
  const dim3 grid(c.kv.n_kv_heads, nsplit, (group * c.m + 15) / 16);
  attn_f32_kernel<HT><<<grid, kF32Waves * 64, lds, st>>>(c.q, c.kv, c.layer, c.m, c.start_pos, c.n_q_heads, nsplit, c.part, c.out);
  return hipGetLastError();
}

hipError_t launch_attn_f32(const AttnCall& c, int nsplit, hipStream_t st) {
  switch (c.kv.head_dim) {
    case 16: return launch_attn_f32_ht<1>(c, nsplit, st);
    case 32: return launch_attn_f32_ht<2>(c, nsplit, st);
    case 48: return launch_attn_f32_ht<3>(c, nsplit, st);
    case 64: return launch_attn_f32_ht<4>(c, nsplit, st);
    case 80: return launch_attn_f32_ht<5>(c, nsplit, st);
    case 96: return launch_attn_f32_ht<6>(c, nsplit, st);
    case 112: return launch_attn_f32_ht<7>(c, nsplit, st);
    case 128: return launch_attn_f32_ht<8>(c, nsplit, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pipesd
