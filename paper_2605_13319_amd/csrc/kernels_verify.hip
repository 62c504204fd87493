// Vocabulary-wide decision of a NAV pass: softmax of the k + 1 logit rows, the accept tests
// u_i < min(1, p_i(d_i)/q_i(d_i)), and the corrected / extra token drawn from max(0, p - q) or
// p_{k+1} (Sec. 2.2: accept what matches, correct the first mismatch; Appendix B: the extra token
// after full acceptance; Sec. 1: the target's output distribution is preserved).
//
// The draw is an integer inverse CDF: weights floor(w * 2^40) are summed as 64-bit integers, which
// is associative, so the parallel scan returns the same index as a sequential one.
#include "common.h"

namespace pipesd {

constexpr int kVThreads = 256;
constexpr int kStatChunks = 64;   // softmax partials per row
constexpr int kScanBlocks = 64;   // workgroups of the CDF scan
constexpr int kHold = 8;          // values a thread holds in registers at once

struct Uniforms {
  float u[kMaxRows];
};

__device__ __forceinline__ unsigned long long shfl_u64(unsigned long long v, int src) {
  unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
  lo = __shfl(lo, src, 64);
  hi = __shfl(hi, src, 64);
  return ((unsigned long long)hi << 32) | lo;
}
// ------------------------------------------------------------------------------------------
// softmax: per (row, chunk) max and sum of exp; p = exp(z - M) / S with M, S merged from the chunk
// partials in index order is formed where it is used (spec_accept_kernel), never written out
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kVThreads) void softmax_stats_kernel(const float* __restrict__ z, int V,
                                                                  float* __restrict__ stats) {
  __shared__ float red[kVThreads / 64];
  const int row = blockIdx.y, c = blockIdx.x;
  const int per = (V + kStatChunks - 1) / kStatChunks;
  const int lo = c * per, hi = min(V, lo + per);
  const float* zr = z + (size_t)row * V;
  // A thread's values stay in registers between the two sweeps where they fit (any vocabulary up to
  // 131072): the logits are read once, all of a thread's loads in flight together.  152 rows of
  // 128256: 41 us with two sweeps over memory.
  const bool held = per <= kHold * kVThreads;
  float v[kHold], mx = -INFINITY;
  if (held) {
#pragma unroll
    for (int j = 0; j < kHold; ++j) {
      const int i = lo + (int)threadIdx.x + j * kVThreads;
      v[j] = i < hi ? zr[i] : -INFINITY;
    }
#pragma unroll
    for (int j = 0; j < kHold; ++j) mx = fmaxf(mx, v[j]);
  } else {
    for (int i = lo + threadIdx.x; i < hi; i += kVThreads) mx = fmaxf(mx, zr[i]);
  }
  mx = fold_wave(mx, LaneMax{});
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  float s = 0.f;
  if (held) {
#pragma unroll
    for (int j = 0; j < kHold; ++j)
      if (lo + (int)threadIdx.x + j * kVThreads < hi) s += expf(v[j] - mx);
  } else {
    for (int i = lo + threadIdx.x; i < hi; i += kVThreads) s += expf(zr[i] - mx);
  }
  s = fold_wave(s, LaneAdd{});
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    stats[((size_t)row * kStatChunks + c) * 2 + 0] = mx;
    stats[((size_t)row * kStatChunks + c) * 2 + 1] = (red[0] + red[1]) + (red[2] + red[3]);
  }
}

hipError_t launch_softmax_stats(const VerifyCall& c, hipStream_t st) {
  dim3 grid(kStatChunks, c.k + 1);
  softmax_stats_kernel<<<grid, kVThreads, 0, st>>>(c.logits_or_p, c.V, c.row_stats);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// decision on probabilities
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ bool accept_test(float p, float q, float u) {
  if (p == 0.f && q == 0.f) return false;  // 0/0 rejects
  const float ratio = p / q;               // correctly rounded fp32 division
  return u < fminf(1.0f, ratio);
}

__device__ __forceinline__ unsigned long long fixed_weight(float p, float q, bool residual) {
  const float w = residual ? fmaxf(0.0f, p - q) : p;
  return (unsigned long long)((double)w * 1099511627776.0);  // floor(w * 2^40), exact
}

// `stats` == nullptr: `p` holds probabilities.  Otherwise `p` holds logits and `stats` the (max,
// sum of exp) chunk partials of softmax_stats_kernel: the probabilities expf(z - M) / S are formed here,
// where they are used, and nowhere else.
// (drafts[0..k-1] and un[0..k] may point into kernel arguments)
//
// Bound by a chain of dependent latencies, not by the 1 MB it reads at a vocabulary of 128256: the
// rows' statistics, the tests, a sweep over one row, the arrival of the other workgroups, the draw.
// Each link asks for all it needs at once, and the draw (find the chunk, then the token in it) is two
// scans by the whole last workgroup.  The chunk sums reach it written through and read past the
// caches, without fences (a device-scope fence writes the whole L2 back), every wave makes the tests for
// itself, and the arrival counter wraps to zero by itself, so that no launch has to clear it in front:
// 9.7 -> 7.8 us on given probabilities at that vocabulary and 8 drafts, and 1.4 for the clearing launch.  With its sums and
// scans on the vector unit (device_lanes.h) calls of the static entry point follow each other every 7.0 us, which is now the
// kernel's time (11.3 before, the host's, whose arguments and stream then came by detours).
__device__ __forceinline__ void spec_accept_body(const float* __restrict__ p, const float* __restrict__ q,
                                                 const float* __restrict__ stats, int k, int V, const int32_t* drafts,
                                                 const float* un, unsigned long long* partial, unsigned* counter,
                                                 int32_t* __restrict__ result, int32_t* __restrict__ result_copy) {
  constexpr int kWaves = kVThreads / 64, kNone = 0x7fffffff;
  __shared__ unsigned long long red[kWaves];
  __shared__ int s_last, s_next;
  __shared__ float s_M[kMaxRows], s_S[kMaxRows];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const bool from_logits = stats != nullptr;
  // operands of the k tests, side by side: lane i of every wave has test i
  static_assert(kMaxRows <= 64, "a lane per test");
  float test_p = 0.f, test_q = 0.f, test_u = 0.f;
  if (lane < k) {
    const size_t at = (size_t)lane * V + drafts[lane];
    test_p = p[at];
    test_q = q[at];
    test_u = un[lane];
  }
  // Row statistics: one wave per row, lane j holding chunk j's (max, sum of exp); the row's max and
  // the rescaled sum are folded across the wave in a fixed butterfly order.  Every workgroup does
  // this for all k + 1 rows itself (one 512-byte load per row).
  static_assert(kStatChunks == 64, "one chunk partial per lane");
  if (from_logits) {
    const int sper = (V + kStatChunks - 1) / kStatChunks;
    const bool have = lane * sper < V;
    constexpr int kRowsPerWave = kMaxRows / kWaves;
    float2 ms[kRowsPerWave];
#pragma unroll
    for (int j = 0; j < kRowsPerWave; ++j) {
      const int row = w + j * kWaves;
      ms[j] = have && row <= k ? *(const float2*)(stats + ((size_t)row * kStatChunks + lane) * 2) : make_float2(-INFINITY, 0.f);
    }
#pragma unroll
    for (int j = 0; j < kRowsPerWave; ++j) {
      const int row = w + j * kWaves;
      if (row > k) break;
      const float M = fold_wave(ms[j].x, LaneMax{});
      const float S = fold_wave(have ? ms[j].y * expf(ms[j].x - M) : 0.f, LaneAdd{});
      if (lane == 0) {
        s_M[row] = M;
        s_S[row] = S;
      }
    }
    __syncthreads();
  }
  bool fails = false;
  if (lane < k) fails = !accept_test(from_logits ? expf(test_p - s_M[lane]) / s_S[lane] : test_p, test_q, test_u);
  const unsigned long long failed = __ballot(fails);  // the tests count in order, up to the first failure
  const int a = failed != 0 ? __ffsll((long long)failed) - 1 : k;
  const bool residual = a < k;
  const float* pr = p + (size_t)a * V;
  const float* qr = q + (size_t)(residual ? a : 0) * V;
  const float row_M = from_logits ? s_M[a] : 0.f, row_S = from_logits ? s_S[a] : 1.f;
  auto prob = [&](float v) -> float { return from_logits ? expf(v - row_M) / row_S : v; };
  // weights of the tokens i0, i0 + step, .. (kHold of them; 0 from `end` on)
  auto weights = [&](int i0, int step, int end, unsigned long long (&out)[kHold]) {
    float pv[kHold], qv[kHold];
#pragma unroll
    for (int j = 0; j < kHold; ++j) {
      const int i = min(i0 + j * step, V - 1);
      pv[j] = pr[i];
      qv[j] = residual ? qr[i] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < kHold; ++j) out[j] = i0 + j * step < end ? fixed_weight(prob(pv[j]), qv[j], residual) : 0ull;
  };

  const int per = (V + kScanBlocks - 1) / kScanBlocks;
  const int lo = blockIdx.x * per, hi = min(V, lo + per);
  unsigned long long s = 0, wt[kHold];
  for (int base = lo; base < hi; base += kVThreads * kHold) {
    weights(base + tid, kVThreads, hi, wt);
#pragma unroll
    for (int j = 0; j < kHold; ++j) s += wt[j];
  }
  s = sum_wave(s);
  if (lane == 0) red[w] = s;
  __syncthreads();
  if (tid == 0) {
    s_next = kNone;
    // written through to memory, acknowledged, then counted in.  (The counter wraps: it is zero again once
    // all workgroups of a launch have arrived, whatever they find.)
    __hip_atomic_store(&partial[blockIdx.x], red[0] + red[1] + red[2] + red[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    s_last = atomicInc(counter, (unsigned)kScanBlocks - 1u) == (unsigned)kScanBlocks - 1u;
  }
  __syncthreads();
  if (!s_last) return;

  // the last workgroup to arrive finishes the draw: lane b of every wave has the sum of chunk b
  static_assert(kScanBlocks == 64, "one chunk sum per lane");
  auto decide = [&](int next) {
    result[0] = a;
    result[1] = next;
    if (result_copy != nullptr) {
      result_copy[0] = a;
      result_copy[1] = next;
    }
  };
  const unsigned long long mine = __hip_atomic_load(&partial[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned long long upto = scan_wave(mine), W = shfl_u64(upto, 63);
  if (W == 0) {
    // every weight truncated to zero: lowest-index maximum of the target row
    if (tid >= 64) return;
    float best = -INFINITY;
    int bi = 0x7fffffff;
    for (int i = tid; i < V; i += 64) {
      const float v = prob(pr[i]);
      if (v > best) { best = v; bi = i; }
    }
    for (int o = 32; o > 0; o >>= 1) {
      const float ob = __shfl_xor(best, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
    }
    if (tid == 0) decide(bi);
    return;
  }
  const unsigned long long ui = (unsigned long long)(un[k] * 16777216.0f);  // floor(u * 2^24)
  const unsigned long long T = (__umul64hi(W, ui) << 40) | ((W * ui) >> 24);
  // chunk whose running total first exceeds T (T < W: there is one, lane 63's total being W)
  const int above = __ffsll((long long)__ballot(upto > T)), b = above > 0 ? above - 1 : kScanBlocks - 1;
  unsigned long long run = shfl_u64(upto, b) - shfl_u64(mine, b);
  const int clo = b * per, chi = min(V, clo + per);
  // The smallest token of the chunk whose running sum exceeds T (the last one if none does): every
  // thread looks through its own tokens, a wave's first finder takes part in the minimum.  Thread 0
  // reports it, so that a result is written whatever the sums are.  (The sums
  // between the tokens count, not only those between the threads: weights of distributions with masses
  // beyond 2^24 wrap.)
  for (int base = clo; base < chi; base += kVThreads * kHold) {
    // thread t has the kHold tokens behind base + t * kHold
    const int i0 = base + tid * kHold;
    weights(i0, 1, chi, wt);
    unsigned long long own = 0;
#pragma unroll
    for (int j = 0; j < kHold; ++j) own += wt[j];
    const unsigned long long inc = scan_wave(own);
    if (lane == 63) red[w] = inc;  // (everybody has read what was there: a barrier lies behind each read)
    __syncthreads();
    unsigned long long at = run + inc - own;  // sum in front of the thread's first token
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) {
      if (ww < w) at += red[ww];
      run += red[ww];
    }
    int found = kNone;
#pragma unroll
    for (int j = 0; j < kHold; ++j) {
      at += wt[j];
      if (at > T) found = min(found, i0 + j);
    }
    const int finder = __ffsll((long long)__ballot(found != kNone));
    if (finder == lane + 1) atomicMin(&s_next, found);
    __syncthreads();
    if (s_next != kNone) break;
  }
  if (tid == 0) decide(min(s_next, chi - 1));
}

__global__ __launch_bounds__(kVThreads) void spec_accept_kernel(const float* __restrict__ p, const float* __restrict__ q,
                                                                const float* __restrict__ stats, int k, int V,
                                                                RowTokens drafts, Uniforms un, unsigned long long* partial,
                                                                unsigned* counter, int32_t* __restrict__ result,
                                                                int32_t* __restrict__ result_copy) {
  spec_accept_body(p, q, stats, k, V, drafts.tok, un.u, partial, counter, result, result_copy);
}

hipError_t launch_spec_accept(const VerifyCall& c, hipStream_t st) {
  Uniforms un;
  for (int i = 0; i < kMaxRows; ++i) un.u[i] = c.u[i];
  spec_accept_kernel<<<kScanBlocks, kVThreads, 0, st>>>(c.logits_or_p, c.q, c.from_logits ? c.row_stats : nullptr, c.k,
                                                        c.V, c.drafts, un, c.scan_partial,
                                                        c.counter, c.result, c.result_copy);
  return hipGetLastError();
}

// The decisions of all clients of a pass in one launch: workgroups (scan block, client).  Client ci
// owns logits rows row_off .. row_off + k of the pass, partial sums [ci][kScanBlocks], counter ci and
// result slots 2 slot, 2 slot + 1; its drafts and uniforms sit at the indices of its rows.  Each client
// is decided by the very code of the single-client kernel.
__global__ __launch_bounds__(kVThreads) void spec_accept_batch_kernel(const float* __restrict__ logits,
                                                                      const float* __restrict__ stats, int V,
                                                                      DecisionBatch b, unsigned long long* partial,
                                                                      unsigned* counter, int32_t* __restrict__ result,
                                                                      int32_t* __restrict__ result_copy) {
  const int ci = blockIdx.y;
  const DecisionClient c = b.c[ci];
  spec_accept_body(logits + (size_t)c.row_off * V, c.q, stats + (size_t)c.row_off * kStatChunks * 2, c.k, V,
                   b.drafts.tok + c.row_off, b.u + c.row_off, partial + (size_t)ci * kScanBlocks, counter + ci,
                   result + 2 * c.slot, result_copy ? result_copy + 2 * c.slot : nullptr);
}

hipError_t launch_spec_accept_batch(const DecisionCall& c, hipStream_t st) {
  if (c.batch.n < 1 || c.batch.n > kMaxPassClients || c.rows < 1 || c.rows > kMaxPassRows) return hipErrorInvalidValue;
  for (int i = 0; i < c.batch.n; ++i) {
    const DecisionClient& d = c.batch.c[i];
    if (d.q == nullptr || d.k < 1 || d.k > kMaxRows - 1 || d.row_off < 0 || d.row_off + d.k + 1 > c.rows || d.slot < 0)
      return hipErrorInvalidValue;
  }
  softmax_stats_kernel<<<dim3(kStatChunks, c.rows), kVThreads, 0, st>>>(c.logits, c.V, c.row_stats);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  spec_accept_batch_kernel<<<dim3(kScanBlocks, c.batch.n), kVThreads, 0, st>>>(
      c.logits, c.row_stats, c.V, c.batch, c.scan_partial, c.counter, c.result, c.result_copy);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// token matching on logits: per (row, chunk) argmax, then one workgroup decides
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kVThreads) void argmax_partial_kernel(const float* __restrict__ z, int V,
                                                                   float* __restrict__ stats) {
  __shared__ float rb[kVThreads / 64];
  __shared__ int ri[kVThreads / 64];
  const int row = blockIdx.y, c = blockIdx.x;
  const int per = (V + kStatChunks - 1) / kStatChunks;
  const int lo = c * per, hi = min(V, lo + per);
  const float* zr = z + (size_t)row * V;
  float best = -INFINITY;
  int bi = 0x7fffffff;
  for (int i = lo + threadIdx.x; i < hi; i += kVThreads) {
    const float v = zr[i];
    if (v > best) { best = v; bi = i; }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const float ob = __shfl_xor(best, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
  }
  if ((threadIdx.x & 63) == 0) { rb[threadIdx.x >> 6] = best; ri[threadIdx.x >> 6] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kVThreads / 64; ++w)
      if (rb[w] > best || (rb[w] == best && ri[w] < bi)) { best = rb[w]; bi = ri[w]; }
    stats[((size_t)row * kStatChunks + c) * 2 + 0] = best;
    stats[((size_t)row * kStatChunks + c) * 2 + 1] = __int_as_float(bi);
  }
}

// one wave per row, lane j holding chunk j's (max, index)
constexpr int kDecideWaves = 16;
__global__ __launch_bounds__(kDecideWaves * 64) void greedy_decide_kernel(const float* __restrict__ stats, int k, int V,
                                                                          RowTokens drafts, int32_t* __restrict__ result,
                                                                          int32_t* __restrict__ result_copy) {
  __shared__ int am[kMaxRows];
  const int per = (V + kStatChunks - 1) / kStatChunks;
  const int lane = threadIdx.x & 63;
  for (int row = threadIdx.x >> 6; row <= k; row += kDecideWaves) {
    const bool have = lane * per < V;
    const float2 st = have ? *(const float2*)(stats + ((size_t)row * kStatChunks + lane) * 2) : make_float2(-INFINITY, 0.f);
    float best = st.x;
    int bi = have ? __float_as_int(st.y) : 0x7fffffff;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float ob = __shfl_xor(best, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
    }
    if (lane == 0) am[row] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int a = 0;
    while (a < k && am[a] == drafts.tok[a]) ++a;
    result[0] = a;
    result[1] = am[a];
    if (result_copy != nullptr) {
      result_copy[0] = a;
      result_copy[1] = am[a];
    }
  }
}

hipError_t launch_greedy_accept(const VerifyCall& c, hipStream_t st) {
  dim3 grid(kStatChunks, c.k + 1);
  argmax_partial_kernel<<<grid, kVThreads, 0, st>>>(c.logits_or_p, c.V, c.row_stats);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  greedy_decide_kernel<<<1, kDecideWaves * 64, 0, st>>>(c.row_stats, c.k, c.V, c.drafts, c.result, c.result_copy);
  return hipGetLastError();
}

}  // namespace pipesd
