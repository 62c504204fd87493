// Row setup, the fp32 rotary step of head sizes the fused one does not take, and KV bookkeeping kernels.
#include "common.h"

namespace pipesd {

// ---------------------------------------------------------------------------------------------
// Row setup: x_r = E[token_r] (fp32 residual stream) and cos/sin(pos_r * theta_i), the angle
// evaluated in fp64 and rounded once (rotary positions; the target forward of Sec. 2.2).
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ void setup_rows_kernel(const T* __restrict__ emb, PassTokens toks, RowMap map, int row0, int m, int d, int half,
                                  const double* __restrict__ theta, float* __restrict__ xres,
                                  float* __restrict__ rope_cs, const float* __restrict__ gain, uint4* xpk,
                                  int act_tiles, float* __restrict__ ssq_out, int ssq_stride,
                                  RowMap* __restrict__ map_dev, TableUpdate update) {
  __shared__ float red[4];
  const int b = blockIdx.x, r = row0 + b;  // (tokens and positions are those of the launch's own rows)
  if (b >= m) return;
  if (map_dev != nullptr && r == 0 && threadIdx.x < kMaxPassRows) {
    map_dev->pos[threadIdx.x] = map.pos[threadIdx.x];
    map_dev->table_off[threadIdx.x] = map.table_off[threadIdx.x];
  }
  if (b == 0 && (int)threadIdx.x < update.n) update.table[update.at[threadIdx.x]] = update.v[threadIdx.x];
  const size_t base = (size_t)toks.tok[b] * d;
  float sq = 0.f;
  for (int j = threadIdx.x; j < d / 8; j += blockDim.x) {
    float v[8], y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      v[i] = load_elem(emb, base + j * 8 + i);
      xres[(size_t)r * d + j * 8 + i] = v[i];
      sq = fmaf(v[i], v[i], sq);
    }
    if (xpk != nullptr) {
#pragma unroll
      for (int i = 0; i < 8; ++i) y[i] = v[i] * gain[j * 8 + i];
      store_act8(xpk, r, j * 8, y, act_tiles);
    }
  }
  for (int i = (d / 8) * 8 + threadIdx.x; i < d; i += blockDim.x) xres[(size_t)r * d + i] = load_elem(emb, base + i);
  if (ssq_out != nullptr) {
    sq = fold_wave(sq, LaneAdd{});
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0) ssq_out[(size_t)r * ssq_stride] = (red[0] + red[1]) + (red[2] + red[3]);
  }
  for (int i = threadIdx.x; i < half; i += blockDim.x) {
    const double ang = (double)map.pos[b] * theta[i];
    rope_cs[((size_t)r * half + i) * 2 + 0] = (float)cos(ang);
    rope_cs[((size_t)r * half + i) * 2 + 1] = (float)sin(ang);
  }
}

hipError_t launch_setup_rows(int dtype, const void* tok_emb, const PassTokens& toks, const RowMap& map, int row0, int m,
                             int d_model, int head_dim, const double* theta, float* xres, float* rope_cs,
                             const float* gain, void* xpk, int act_tiles, float* ssq_out, int ssq_stride,
                             RowMap* map_dev, const TableUpdate& update, hipStream_t st) {
  if (dtype == PIPESD_F32)
    setup_rows_kernel<float><<<m, 256, 0, st>>>((const float*)tok_emb, toks, map, row0, m, d_model, head_dim / 2, theta, xres,
                                                rope_cs, nullptr, nullptr, 0, nullptr, 0, map_dev, update);
  else
    setup_rows_kernel<uint16_t><<<m, 256, 0, st>>>((const uint16_t*)tok_emb, toks, map, row0, m, d_model, head_dim / 2, theta,
                                                   xres, rope_cs, gain, (uint4*)xpk, act_tiles, ssq_out, ssq_stride,
                                                   map_dev, update);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// fp32 path, head_dim not a multiple of 16 (else the QKV product's epilogue does this)
// ---------------------------------------------------------------------------------------------
// rotate q and k, store q to the query buffer and k, v to the paged cache (fp32 cache)
__global__ void rope_append_f32_kernel(const float* __restrict__ qkv, int m, int start_pos, int layer, int n_q_heads,
                                       KvView kv, const float* __restrict__ rope_cs, float* __restrict__ qbuf) {
  const int h = kv.head_dim, half = h / 2;
  const int n_heads = n_q_heads + 2 * kv.n_kv_heads;
  const int ld = n_heads * h;
  const int r = blockIdx.y, hd = blockIdx.x;
  float* kvp = (float*)kv.pool;
  for (int i = threadIdx.x; i < half; i += blockDim.x) {
    const float a = qkv[(size_t)r * ld + hd * h + i], b = qkv[(size_t)r * ld + hd * h + i + half];
    const float c = rope_cs[((size_t)r * half + i) * 2], s = rope_cs[((size_t)r * half + i) * 2 + 1];
    if (hd < n_q_heads) {
      qbuf[(size_t)r * n_q_heads * h + hd * h + i] = a * c - b * s;
      qbuf[(size_t)r * n_q_heads * h + hd * h + i + half] = b * c + a * s;
    } else if (hd < n_q_heads + kv.n_kv_heads) {
      const int kvh = hd - n_q_heads;
      kvp[k_index(kv, layer, start_pos + r, kvh, i)] = a * c - b * s;
      kvp[k_index(kv, layer, start_pos + r, kvh, i + half)] = b * c + a * s;
    } else {
      const int kvh = hd - n_q_heads - kv.n_kv_heads;
      kvp[v_index(kv, layer, start_pos + r, kvh, i)] = a;
      kvp[v_index(kv, layer, start_pos + r, kvh, i + half)] = b;
    }
  }
}

hipError_t launch_rope_append_f32(const float* qkv, int m, int start_pos, int layer, int n_q_heads, const KvView& kv,
                                  const float* rope_cs, float* qbuf, hipStream_t st) {
  dim3 grid(n_q_heads + 2 * kv.n_kv_heads, m);
  rope_append_f32_kernel<<<grid, 64, 0, st>>>(qkv, m, start_pos, layer, n_q_heads, kv, rope_cs, qbuf);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// In-place KV truncation: the rows of the rejected drafts are cleared in every layer, so nothing
// of a rejected suffix survives in the cache (rollback to the last accepted token, Appendix B).
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ void kv_trim_kernel(KvView kv, int first_pos, int k, const int32_t* __restrict__ result) {
  const int a = result[0];
  const int j = blockIdx.x;  // draft row index 1..k -> position first_pos + j
  const int layer = blockIdx.y;
  if (j + 1 <= a) return;    // draft j+1 accepted
  const int pos = first_pos + j + 1;
  T* p = (T*)kv.pool;
  const int kvd = kv.n_kv_heads * kv.head_dim;
  for (int i = threadIdx.x; i < kvd; i += blockDim.x) {
    const int kvh = i / kv.head_dim, e = i % kv.head_dim;
    p[k_index(kv, layer, pos, kvh, e)] = (T)0;
    p[v_index(kv, layer, pos, kvh, e)] = (T)0;
  }
}

hipError_t launch_kv_trim(int dtype, const KvView& kv, int n_layers, int first_pos, int k, const int32_t* result,
                          hipStream_t st) {
  if (k <= 0) return hipSuccess;
  dim3 grid(k, n_layers);
  if (dtype == PIPESD_F32)
    kv_trim_kernel<float><<<grid, 256, 0, st>>>(kv, first_pos, k, result);
  else
    kv_trim_kernel<uint16_t><<<grid, 256, 0, st>>>(kv, first_pos, k, result);
  return hipGetLastError();
}

// grid (draft rows of the longest client, layers, clients)
template <typename T>
__global__ void kv_trim_batch_kernel(KvView kv, TrimBatch b, const int32_t* __restrict__ result) {
  const TrimClient c = b.c[blockIdx.z];
  const int a = result[2 * c.slot];
  const int j = blockIdx.x;
  const int layer = blockIdx.y;
  if (j >= c.k || j + 1 <= a) return;
  kv.table += c.table_off;
  const int pos = c.first_pos + j + 1;
  T* p = (T*)kv.pool;
  const int kvd = kv.n_kv_heads * kv.head_dim;
  for (int i = threadIdx.x; i < kvd; i += blockDim.x) {
    const int kvh = i / kv.head_dim, e = i % kv.head_dim;
    p[k_index(kv, layer, pos, kvh, e)] = (T)0;
    p[v_index(kv, layer, pos, kvh, e)] = (T)0;
  }
}

hipError_t launch_kv_trim_batch(int dtype, const KvView& kv, int n_layers, const TrimBatch& b, const int32_t* result,
                                hipStream_t st) {
  if (b.n < 1 || b.n > kMaxPassClients) return hipErrorInvalidValue;
  int max_k = 0;
  for (int i = 0; i < b.n; ++i) max_k = b.c[i].k > max_k ? b.c[i].k : max_k;
  if (max_k <= 0) return hipSuccess;
  dim3 grid(max_k, n_layers, b.n);
  if (dtype == PIPESD_F32)
    kv_trim_batch_kernel<float><<<grid, 256, 0, st>>>(kv, b, result);
  else
    kv_trim_batch_kernel<uint16_t><<<grid, 256, 0, st>>>(kv, b, result);
  return hipGetLastError();
}

constexpr int kTableEntries = 128;  // per launch (a prompt of 2048 tokens in one)
struct TableEntries {
  int32_t v[kTableEntries];
};
__global__ void set_table_kernel(int32_t* table, int first, TableEntries e, int n) {
  if ((int)threadIdx.x < n) table[first + threadIdx.x] = e.v[threadIdx.x];
}

hipError_t launch_set_table(int32_t* table, int first, const int32_t* entries, int n, hipStream_t st) {
  for (int i = 0; i < n; i += kTableEntries) {
    TableEntries e;
    const int c = (n - i < kTableEntries) ? (n - i) : kTableEntries;
    for (int j = 0; j < kTableEntries; ++j) e.v[j] = j < c ? entries[i + j] : 0;
    set_table_kernel<<<1, kTableEntries, 0, st>>>(table, first + i, e, c);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

__global__ void chain_step_kernel(int32_t* result, int32_t* result_copy, int k, int guess, const int32_t* alive_in,
                                  int32_t* alive_out) {
  if (threadIdx.x != 0) return;
  const bool alive = alive_in == nullptr || *alive_in != 0;
  if (!alive) {
    result[0] = result[1] = -1;
    if (result_copy != nullptr) result_copy[0] = result_copy[1] = -1;
  }
  if (alive_out != nullptr) *alive_out = (alive && result[0] == k && result[1] == guess) ? 1 : 0;
}

hipError_t launch_chain_step(int32_t* result, int32_t* result_copy, int k, int guess, const int32_t* alive_in,
                             int32_t* alive_out, hipStream_t st) {
  chain_step_kernel<<<1, 64, 0, st>>>(result, result_copy, k, guess, alive_in, alive_out);
  return hipGetLastError();
}

}  // namespace pipesd
