// GEMM for passes of more than 32 rows (batched verification of several clients, prompt ingestion).
//
// At this many rows the activations of a K slice no longer fit a wave's registers, and spreading the
// rows over workgroups that re-read the weights from the L2 (the narrow kernel's way) moves many
// times the weights through it.  Here a workgroup of eight waves (two per SIMD) multiplies a tile of
// rows x columns whose operands reach the matrix cores through LDS, without passing through registers
// on the way there: every wave asks for its share of a k-step's fragments (the tile's weight fragments
// and its row tiles' activation fragments, hi and lo) with loads that write straight into LDS, into a
// ring of up to five k-steps.  ActPack and the re-tiled weights are already in the lane order the
// matrix cores consume, so a fragment is 64 lanes x 16 bytes, copied as it is, and an operand advances
// by a constant from k-step to k-step: a request is a per-lane offset that never changes and a scalar
// base that moves on.
//
// A k-step of the loop: wait until this wave's share of the next k-step has landed (loads return in
// order), one workgroup barrier, then the current k-step's products in groups of four with, in front of
// each group, a part of the next k-step's operand reads (into the other half of the operand registers)
// and of the requests, which go into the buffer of the k-step before the current one.  Issued all at
// once behind the barrier the reads of the eight waves fill the LDS queue and hold up the products
// behind them (2048 rows, 28672 x 4096: 814 against 743 us).  Wave (wm, wn) owns row tiles r * WM + wm,
// r < RT, x four n-tiles.  What LDS has to deliver per product falls with the wave's tile: 4 x 4 tiles
// take 12 KB per 32 products, 2 x 4 take 8 KB per 16.  Row tiles past the pass are neither read nor
// multiplied.
//
// What bounds it: the matrix cores' rate in a loop of this form, 1.5 PFLOP/s of issued bf16 products
// (hi and lo halves counted; measured with the same operand reads, barriers and copies but nothing
// else; a large library product of this device reaches 1.5 - 1.6), and for passes of few row tiles the
// weights' way from memory.  Issued rates: 2048 rows 1.24 - 1.36 PFLOP/s (gate/up of the 8B shape 708 -
// 778 us in several sessions, the matrix cores busy in 67 % of the cycles; 128 rows at a time with one row
// tile x four n-tiles per wave it took 16 x 83), 152 rows 0.91 (83 us, before 108), 68 rows 3.6 TB/s of
// weights (65 us, before 78; with the weights held in the caches 49).
//
// Results are bit-identical to the narrow kernel's, row by row: K is cut into the same W * P slices
// of 512 columns, every slice is accumulated from zero in the same k-step order (hi half, then lo
// half of the activations), slices p*W + w are added in the order p = 0..P-1 and the W sums in the
// order w = 0..W-1, starting from zero.  Two ways to get enough workgroups:
//  * WHOLE: a workgroup walks all slices of its tile and finishes it itself (epilogue from the
//    accumulators; RMSNorm's rstd per row comes from a small kernel in front: computed by every
//    workgroup it took 6 - 8 us of each).  Registers hold the slice being accumulated and one more sum per output; with
//    phases (P > 1) that is the role's running sum, and the total of the roles waits in memory, read
//    and written once per role;
//  * split: workgroup (tile, w) walks the P slices of role w only and leaves its running sum in a
//    workspace; a second small kernel adds the W sums in order and runs the epilogue.
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "device_dma.h"
#include "device_gemm.h"
#include "lds_limit.h"

namespace pipesd {

constexpr int kWideWaves = 8;
constexpr int kWideMaxRoles = 8;  // W <= 8 (launch shape)
// Tile shapes: WM x WN waves of RT x 4 tiles
constexpr int wide_kstep_frags(int wm, int wn, int rt) { return wn * 4 + 2 * wm * rt; }
// k-steps held in LDS: as many as 160 KB take, up to five (one being read, three on their way, one freed
// by the barrier that the next request goes into); more gave nothing
constexpr int wide_ring(int wm, int wn, int rt) {
  const int fit = 160 / wide_kstep_frags(wm, wn, rt);
  return fit < 5 ? fit : 5;
}
constexpr size_t wide_lds_bytes(int wm, int wn, int rt) { return (size_t)wide_ring(wm, wn, rt) * wide_kstep_frags(wm, wn, rt) * 1024; }

struct WideArgs {
  f32x4* ws;          // split: [W][ntiles][row tiles][64] running sums of role w; whole with phases: [ntiles][row tiles][64] totals
  const float* rstd;  // per row (products with a fused norm)
  int ncg, nrb;       // column groups, row blocks
  int row_tiles;      // live row tiles of the pass
  int block_tiles;    // row tiles per row block (the last one may have fewer)
  int rchunk;         // row blocks that are walked next to each other
};

// f(integral_constant<int, n>) for the run-time n in 0..N
template <int N, class F>
__device__ __forceinline__ void wide_dispatch_count(int n, F& f) {
  if constexpr (N == 0) {
    f(std::integral_constant<int, 0>{});
  } else {
    if (n == N) f(std::integral_constant<int, N>{});
    else wide_dispatch_count<N - 1>(n, f);
  }
}

// EPI: the epilogue of a whole walk (a split one has none: kEpiAny).  One kernel with all four behind branches at run time took,
// us (that / this): 8B gate/up 33 rows 54.6 / 53.9, QKV 333 rows 62.0 / 60.9 and 2047 rows 196 / 192; 3584 columns gate/up 33 rows
// 71.3 / 69.3; 1B gate/up 96 rows 30.3 / 29.9.
template <int WM, int WN, int RT, bool WHOLE, bool P1, int EPI>
__global__ __launch_bounds__(kWideWaves * 64) void gemm_wide_kernel(GemmArgs a, WideArgs x) {
  static_assert(WM * WN == kWideWaves, "eight waves");
  extern __shared__ float lds_f[];
  constexpr int CT = WN * 4, TILES = WM * RT;         // n-tiles and row tiles of the workgroup
  constexpr int KF = wide_kstep_frags(WM, WN, RT);    // fragments per k-step: the CT weight fragments, then (row tile, half)
  constexpr int NW_ = CT / kWideWaves;                // weight fragments this wave requests per k-step
  constexpr int NA = (2 * TILES + kWideWaves - 1) / kWideWaves;  // activation fragments
  constexpr int NPER = NW_ + NA;
  constexpr int RG = wide_ring(WM, WN, RT), kBuf = KF * 1024, kRing = RG * kBuf;
  static_assert(CT % kWideWaves == 0 && RG >= 4, "weight fragments are dealt evenly");
  char* ring = (char*)lds_f;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (waves w and w + 4 share a SIMD: they get different row tiles, so that an odd number spreads evenly)
  const int wm = w / WN, wn = w % WN;
  // Tiles are dealt so that a chiplet (workgroups b, b + 8, ..) walks a contiguous run of them, in the
  // order (chunk of row blocks, column group, role, row block): workgroups that run side by side on
  // a chiplet share operands through its L2.
  const int nrole = WHOLE ? 1 : a.W, ntask = x.ncg * x.nrb * nrole;
  const int per_xcd = (ntask + 7) / 8, task = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || task >= ntask) return;
  const int chunk = task / (x.rchunk * x.ncg * nrole), in = task - chunk * x.rchunk * x.ncg * nrole;
  const int rc = min(x.rchunk, x.nrb - chunk * x.rchunk);  // row blocks of this chunk
  const int rb = chunk * x.rchunk + in % rc, cr = in / rc, role = cr % nrole, cg = cr / nrole;
  const int rt0 = rb * x.block_tiles, live = min(x.block_tiles, x.row_tiles - rt0);  // row tiles of this workgroup
  const int nsl = (WHOLE ? a.W : 1) * a.P;  // slices this workgroup walks
  const int kslice0 = WHOLE ? 0 : role;     // first slice of the walk

  // requests: per-lane offsets that stay, scalar bases that move on by a k-step
  unsigned voff[NPER];
#pragma unroll
  for (int i = 0; i < NPER; ++i) {
    if (i < NW_) {
      const int t = min(cg * CT + w + kWideWaves * i, a.ntiles - 1) - cg * CT;
      voff[i] = (unsigned)(t * a.kst) * 1024u + lane * 16u;
    } else {
      const int e = min(w + kWideWaves * (i - NW_), 2 * live - 1);  // (past the pass: a fragment that is there, never read)
      voff[i] = (unsigned)e * 1024u + lane * 16u;
    }
  }
  const size_t astep = (size_t)a.act_tiles * 2 * 1024;
  const char* wbase = (const char*)a.wp + ((size_t)cg * CT * a.kst + (size_t)kslice0 * 16) * 1024;
  const char* abase = (const char*)a.actp + (size_t)rt0 * 2 * 1024 + (size_t)kslice0 * 16 * astep;
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)ring;
  auto request_one = [&](int buf, int i) {  // this wave's i-th fragment of the next k-step, into the ring at byte offset buf
    const int f = i < NW_ ? w + kWideWaves * i : CT + min(w + kWideWaves * (i - NW_), 2 * TILES - 1);
    lds_dma16(i < NW_ ? wbase : abase, voff[i], lds0 + (unsigned)(buf + f * 1024));  // (a 1 KB fragment)
  };
  // the requests have covered a slice: move to the next slice of the walk (slice p*W + w follows
  // (p-1)*W + w; role w + 1 follows role w); past the end of the walk, to the last slice again
  int rq_j = 0, rq_p = 0;
  auto request_turn = [&]() {
    int dsl = 0;  // slices from the one just requested to the next
    if (rq_j + 1 < nsl) {
      dsl = a.W;
      if constexpr (WHOLE) {
        if (rq_p + 1 == a.P) dsl = 1 - (a.P - 1) * a.W;
      }
    }
    ++rq_j;
    rq_p = rq_p + 1 == a.P ? 0 : rq_p + 1;
    const ptrdiff_t dk = (ptrdiff_t)(dsl - 1) * 16;  // (the bases are already one slice further)
    wbase += dk * 1024;
    abase += dk * (ptrdiff_t)astep;
  };
  // acc: the slice being accumulated; sum: the roles' total (WHOLE, P == 1) or this role's running sum
  f32x4 acc[4][RT], sum[4][RT];
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[n][r] = sum[n][r] = zero;
  u32x4 wf[2][4], af[2][RT][2];
  const char* lw = ring + (wn * 4 * 64 + lane) * 16;  // this lane's 16 bytes of the wave's first weight fragment
  const char* la = ring + ((CT + wm * 2) * 64 + lane) * 16;  // and of its first activation fragment

  int rq_stage = 0;  // k-steps of the slice being requested that are under way
  auto request_done = [&]() {
    wbase += 1024;
    abase += astep;
    if (++rq_stage == 16) {
      rq_stage = 0;
      request_turn();
    }
  };
#pragma unroll
  for (int b = 0; b < RG - 1; ++b) {
#pragma unroll
    for (int i = 0; i < NPER; ++i) request_one(b * kBuf, i);
    request_done();
  }
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NPER * (RG - 2)) : "memory");
  __builtin_amdgcn_s_barrier();

  int rd = 0, wr = kRing - kBuf;  // k-step being read, and the one to be requested into (byte offsets in the ring)
  // where the role totals of a walk with phases wait
  auto tot = [&](int t, int r) { return x.ws + ((size_t)t * x.row_tiles + rt0 + r * WM + wm) * 64 + lane; };
  auto walk = [&](auto lrc) {
    constexpr int LR = decltype(lrc)::value;
    constexpr int NR = 4 + 2 * LR;  // operand reads of a k-step: weights, then (row tile, half)
    auto read_one = [&](int q, int slot) {
      if (q < 4) wf[slot][q] = *(const u32x4*)(lw + rd + q * 1024);
      else af[slot][(q - 4) >> 1][q & 1] = *(const u32x4*)(la + rd + ((q - 4) >> 1) * WM * 2048 + (q & 1) * 1024);
    };
    if constexpr (LR > 0) {
#pragma unroll
      for (int q = 0; q < NR; ++q) read_one(q, 0);
    }
    int p = 0, wj = 0;
    for (int j = 0; j < nsl; ++j) {
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        // The next k-step has landed for every wave, and nobody reads the one before the current one
        // any more (its products have been issued): its buffer takes the next request.
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NPER * (RG - 3)) : "memory");
        __builtin_amdgcn_s_barrier();
        rd = rd == kRing - kBuf ? 0 : rd + kBuf;
        constexpr int G = LR > 0 ? 2 * LR : 1;           // groups of four products
        constexpr int GR = LR > 1 ? G - G / 4 : 1;       // reads go with the first GR of them
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
#pragma unroll
          for (int i = 0; i < NPER; ++i)
            if (i * G / NPER == gi) request_one(wr, i);
          if constexpr (LR > 0) {
            if (gi < GR) {
#pragma unroll
              for (int q = gi * NR / GR; q < (gi + 1) * NR / GR; ++q) read_one(q, (s + 1) & 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            const int r = gi >> 1, hl = gi & 1;
            const bf16x8 b = as_bf16x8(af[s & 1][r][hl]);
#pragma unroll
            for (int n = 0; n < 4; ++n)
              acc[n][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wf[s & 1][n]), b, s == 0 && hl == 0 ? zero : acc[n][r], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        wr = wr == kRing - kBuf ? 0 : wr + kBuf;
        request_done();
      }
      // The slice is complete.  (The last products may have been issued in another basic block, where
      // the compiler pads no wait states for the adds below: spell them out.)
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int r = 0; r < LR; ++r) {
          if constexpr (P1 && WHOLE) sum[n][r] = sum[n][r] + acc[n][r];  // (zero + first role)
          else if constexpr (P1) sum[n][r] = acc[n][r];
          else sum[n][r] = p == 0 ? acc[n][r] : sum[n][r] + acc[n][r];
        }
      if constexpr (!P1) {
        if (++p == a.P) {
          p = 0;
          if constexpr (WHOLE) {  // a role is complete: into the total (nobody else touches these)
            // (an n-tile's totals asked for before its first store: behind a store each would wait by itself)
#pragma unroll
            for (int n = 0; n < 4; ++n) {
              const int t = cg * CT + wn * 4 + n;
              if (t < a.ntiles) {
                f32x4 old[LR > 0 ? LR : 1];
#pragma unroll
                for (int r = 0; r < LR; ++r) old[r] = wj == 0 ? zero : *tot(t, r);
#pragma unroll
                for (int r = 0; r < LR; ++r) {
                  sum[n][r] = old[r] + sum[n][r];
                  if (wj + 1 < a.W) *tot(t, r) = sum[n][r];
                }
              }
            }
            ++wj;
          }
        }
      }
    }
  };
  {
    int lr = 0;  // this wave's live row tiles
#pragma unroll
    for (int r = 0; r < RT; ++r) lr += (r * WM + wm < live) ? 1 : 0;
    wide_dispatch_count<RT>(lr, walk);
  }
  // the requests past the end of the walk must have landed before the workgroup gives its LDS back
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if constexpr (WHOLE) {
    // What the epilogue reads is asked for before its first store: behind the stores of an earlier tile every
    // load would wait by itself.
    const int t0 = cg * CT + wn * 4;
    const int c = lane & 15;
    float rstd[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) rstd[r] = x.rstd != nullptr ? x.rstd[min((rt0 + r * WM + wm) * 16 + c, a.m - 1)] : 1.0f;
    constexpr bool resid = EPI == EPI_RESID;
#pragma unroll
    for (int n = 0; n < 4; ++n) {  // (an n-tile at a time: registers)
      ResidPre pre[RT];
      if constexpr (resid) {
#pragma unroll
        for (int r = 0; r < RT; ++r) pre[r] = resid_pre(a, t0 + n, (rt0 + r * WM + wm) * 16 + c, lane);
      }
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const int lt = r * WM + wm;
        if (t0 + n < a.ntiles && lt < live)
          epilogue_quad<false, EPI>(a, t0 + n, (rt0 + lt) * 16 + c, lane, sum[n][r], rstd[r], resid, pre[r]);
      }
    }
  } else {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int t = cg * CT + wn * 4 + n;
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const int lt = r * WM + wm, rt = rt0 + lt;
        if (t < a.ntiles && lt < live) x.ws[(((size_t)role * a.ntiles + t) * x.row_tiles + rt) * 64 + lane] = sum[n][r];
      }
    }
  }
}

// rstd of every row of the pass, one wave per row, in the narrow kernel's order: lane sums of the partial
// sums j = lane, lane + 64, .., then the xor butterfly 32, 16, .., 1.  (Latency only: with eight rows per
// wave, whose butterflies wait for each other, it took 7 us instead of 4.6.)
__global__ __launch_bounds__(256) void wide_rstd_kernel(const float* __restrict__ ssq, int stride, int parts, int m, float k, float eps,
                                                        float* __restrict__ rstd) {
  const int lane = threadIdx.x & 63, row = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (row >= m) return;
  float v[kSsqPerLane];
#pragma unroll
  for (int j4 = 0; j4 < kSsqPerLane; ++j4) v[j4] = ssq[(size_t)row * stride + min(lane + 64 * j4, parts - 1)];
  float t = lane < parts ? v[0] : 0.f;
#pragma unroll
  for (int j4 = 1; j4 < kSsqPerLane; ++j4) t += lane + 64 * j4 < parts ? v[j4] : 0.f;
  t = fold_wave(t, LaneAdd{});
  if (lane == 0) rstd[row] = 1.0f / sqrtf(t / k + eps);
}

// split mode, second half: add the W running sums of every 16 x 16 tile in the order w = 0..W-1 and
// finish it.  Workgroup (4 n-tiles, row tile), one tile per wave; all W sums are requested at once.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_wide_finish_kernel(GemmArgs a, WideArgs x) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int rt = (int)blockIdx.y;
  const int t = (int)blockIdx.x * 4 + w;
  if (t >= a.ntiles) return;
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  const int row = rt * 16 + (lane & 15);
  f32x4 pv[kWideMaxRoles];
#pragma unroll
  for (int ww = 0; ww < kWideMaxRoles; ++ww) pv[ww] = x.ws[(((size_t)min(ww, a.W - 1) * a.ntiles + t) * x.row_tiles + rt) * 64 + lane];
  // (the residual epilogue's operands travel with the sums)
  ResidPre pre{};
  constexpr bool resid = EPI == EPI_RESID;
  if constexpr (resid) pre = resid_pre(a, t, row, lane);
  const float rstd = x.rstd != nullptr ? x.rstd[min(row, a.m - 1)] : 1.0f;
  f32x4 v = zero;
#pragma unroll
  for (int ww = 0; ww < kWideMaxRoles; ++ww) v = ww < a.W ? v + pv[ww] : v;
  epilogue_quad<false, EPI>(a, t, row, lane, v, rstd, resid, pre);
}

// ------------------------------------------------------------------------------------------------
// launch shape
// ------------------------------------------------------------------------------------------------
template <int WM, int WN, int RT, bool WHOLE, bool P1, int EPI>
static hipError_t launch_wide_kernel(const GemmArgs& a, const WideArgs& x, int grid, bool timed, hipEvent_t e0,
                                     hipEvent_t e1, hipStream_t st) {
  constexpr size_t lds = wide_lds_bytes(WM, WN, RT);
  static std::atomic<uint64_t> lds_allowed;
  const hipError_t e = allow_lds(lds_allowed, (const void*)gemm_wide_kernel<WM, WN, RT, WHOLE, P1, EPI>, lds);
  if (e != hipSuccess) return e;
  // start of the first kernel of the product, end of the last
  if (timed)
    hipExtLaunchKernelGGL((gemm_wide_kernel<WM, WN, RT, WHOLE, P1, EPI>), dim3(grid), dim3(kWideWaves * 64), (uint32_t)lds, st, e0,
                          WHOLE ? e1 : nullptr, 0, a, x);
  else
    gemm_wide_kernel<WM, WN, RT, WHOLE, P1, EPI><<<grid, kWideWaves * 64, lds, st>>>(a, x);
  return hipGetLastError();
}

hipError_t launch_gemm_wide(const GemmCall& c, GemmArgs a, hipStream_t st) {
  const int n_cu = device_cu_count();
  if (n_cu <= 0) return hipErrorUnknown;
  if (c.act_tiles < 8 || a.K % 512 != 0 || a.W > kWideMaxRoles) return hipErrorInvalidValue;
  const WidePlan p = wide_plan(c.N, c.K, (c.m + 15) / 16, n_cu, c.wide_ws ? c.wide_ws_bytes : 0);
  if (p.ct == 0) return hipErrorInvalidValue;
  const bool timed = c.ev_start != nullptr && c.ev_stop != nullptr;
  hipEvent_t e0 = timed ? c.ev_start : nullptr;
  const hipEvent_t e1 = timed ? c.ev_stop : nullptr;
  if (a.ssq_in != nullptr) {
    if (c.rstd == nullptr) return hipErrorInvalidValue;
    const dim3 rgrid((c.m + 3) / 4);
    if (timed)
      hipExtLaunchKernelGGL(wide_rstd_kernel, rgrid, dim3(256), 0, st, e0, nullptr, 0, a.ssq_in, a.ssq_stride, a.ssq_parts, c.m,
                            (float)a.K, a.eps, c.rstd);
    else
      wide_rstd_kernel<<<rgrid, 256, 0, st>>>(a.ssq_in, a.ssq_stride, a.ssq_parts, c.m, (float)a.K, a.eps, c.rstd);
    e0 = nullptr;
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  WideArgs x{};
  x.ws = (f32x4*)c.wide_ws;
  x.rstd = a.ssq_in != nullptr ? c.rstd : nullptr;
  x.ncg = (a.ntiles + p.ct - 1) / p.ct;
  x.nrb = p.nrb;
  x.row_tiles = (c.m + 15) / 16;
  x.block_tiles = p.block_tiles;
  x.rchunk = std::min(p.nrb, 8);
  const int ntask = x.ncg * x.nrb * (p.whole ? 1 : a.W), grid = (ntask + 7) / 8 * 8;
  auto go = [&](auto wm, auto wn, auto rt) -> hipError_t {
    constexpr int WM = decltype(wm)::value, WN = decltype(wn)::value, RT = decltype(rt)::value;
    if (!p.whole) {
      if (a.P == 1) return launch_wide_kernel<WM, WN, RT, false, true, kEpiAny>(a, x, grid, timed, e0, e1, st);
      return launch_wide_kernel<WM, WN, RT, false, false, kEpiAny>(a, x, grid, timed, e0, e1, st);
    }
    auto whole = [&](auto epi) {
      constexpr int EPI = decltype(epi)::value;
      if (a.P == 1) return launch_wide_kernel<WM, WN, RT, true, true, EPI>(a, x, grid, timed, e0, e1, st);
      return launch_wide_kernel<WM, WN, RT, true, false, EPI>(a, x, grid, timed, e0, e1, st);
    };
    switch (a.epi) {
      case EPI_STORE: return whole(std::integral_constant<int, EPI_STORE>{});
      case EPI_RESID: return whole(std::integral_constant<int, EPI_RESID>{});
      case EPI_SWIGLU: return whole(std::integral_constant<int, EPI_SWIGLU>{});
      default: return whole(std::integral_constant<int, EPI_QKV>{});
    }
  };
  using std::integral_constant;
  hipError_t e = hipErrorInvalidValue;
  if (p.ct == 16 && p.rt == 4) e = go(integral_constant<int, 2>{}, integral_constant<int, 4>{}, integral_constant<int, 4>{});
  else if (p.ct == 16 && p.rt == 3) e = go(integral_constant<int, 2>{}, integral_constant<int, 4>{}, integral_constant<int, 3>{});
  else if (p.ct == 16 && p.rt == 2) e = go(integral_constant<int, 2>{}, integral_constant<int, 4>{}, integral_constant<int, 2>{});
  else if (p.ct == 8 && p.rt == 3) e = go(integral_constant<int, 4>{}, integral_constant<int, 2>{}, integral_constant<int, 3>{});
  else if (p.ct == 8 && p.rt == 2) e = go(integral_constant<int, 4>{}, integral_constant<int, 2>{}, integral_constant<int, 2>{});
  else if (p.ct == 8 && p.rt == 1) e = go(integral_constant<int, 4>{}, integral_constant<int, 2>{}, integral_constant<int, 1>{});
  if (e != hipSuccess || p.whole) return e;
  const dim3 fgrid((a.ntiles + 3) / 4, x.row_tiles);
  auto finish = [&](auto kernel) {
    if (timed)
      hipExtLaunchKernelGGL(kernel, fgrid, dim3(256), 0, st, nullptr, e1, 0, a, x);
    else
      kernel<<<fgrid, 256, 0, st>>>(a, x);
  };
  switch (a.epi) {
    case EPI_STORE: finish(gemm_wide_finish_kernel<EPI_STORE>); break;
    case EPI_RESID: finish(gemm_wide_finish_kernel<EPI_RESID>); break;
    case EPI_SWIGLU: finish(gemm_wide_finish_kernel<EPI_SWIGLU>); break;
    default: finish(gemm_wide_finish_kernel<EPI_QKV>); break;
  }
  return hipGetLastError();
}

}  // namespace pipesd
