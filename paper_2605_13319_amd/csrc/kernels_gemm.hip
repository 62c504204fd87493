// Per-GEMM kernel of the NAV pass: one launch per projection (used for the LM head, for passes with
// more than 16 rows, and for shapes the fused layer kernel does not take).  The device code lives in
// device_gemm.h.
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "device_gemm.h"

namespace pipesd {

// EPI (the projection's epilogue) is a template parameter: every projection of a layer is a kernel
// of its own name, with only its own epilogue's code and registers.
// P1 says that every wave has a single K slice (no phases); ONE that there are phases and that no team
// has more than one tile.
// NR, NL, SHUF: see gemm_body.
template <int KSTEPS, bool NT, int EPI, bool P1, bool ONE = false, int NR = 2, int NL = kSsqPerLane, bool SHUF = false>
__global__ __launch_bounds__(512) void gemm_bf16_kernel(GemmArgs a) {
  extern __shared__ float lds[];
  if (a.gate != nullptr && *a.gate == 0) return;  // (uniform: a round of a chain that does not run)
  const int w = threadIdx.x >> 6;
  // One team per workgroup: all W waves of the workgroup.  With rt row tiles the workgroups b,
  // b + 8, .. b + 8 (rt - 1) form a group on the same tiles (16 rows of the pass each): workgroups
  // are dealt to the 8 chiplets round robin, so a group shares an L2 and the weights cross the
  // memory interface once.
  const int b = (int)blockIdx.x, rt = a.row_tiles;
  TeamPos tp{(b / (8 * rt)) * 8 + (b & 7), (int)gridDim.x / rt, w, 0, true};
  tp.row_base = ((b >> 3) % rt) * 16;
  u32x4 af[KSTEPS];
  gemm_body<1, KSTEPS, false, NT, EPI, P1, ONE, NR, NL, SHUF>(a, tp, 1, a.W, lds, af);
}

// ------------------------------------------------------------------------------------------------
// launch shape
// ------------------------------------------------------------------------------------------------
int device_cu_count() {
  static int n_cu = 0;
  if (n_cu == 0) {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
    n_cu = prop.multiProcessorCount;
  }
  return n_cu;
}

hipError_t launch_gemm_bf16(const GemmCall& c, hipStream_t st) {
  const int n_cu = device_cu_count();
  if (n_cu <= 0) return hipErrorUnknown;
  if (c.m < 1 || c.m > kMaxPromptRows || c.K % 512 != 0 || c.act_tiles * 16 < c.m) return hipErrorInvalidValue;
  const int row_tiles = (c.m + 15) / 16;
  const GemmPlan p = gemm_narrow_plan(c.N, c.K, row_tiles, n_cu);
  GemmArgs a{};
  a.wp = (const u32x4*)c.wp;
  a.actp = (const u32x4*)c.actp;
  a.ssq_in = c.ssq_in;
  a.ssq_parts = c.ssq_parts;
  a.ssq_stride = c.ssq_stride;
  a.out = c.out;
  a.res_in = c.res_in;
  a.outp = (u32x4*)c.outp;
  a.gain_next = c.gain_next;
  a.ssq_out = c.ssq_out;
  a.rope_cs = c.rope_cs;
  a.rows = c.rows;
  a.kv = c.kv;
  a.m = c.m;
  a.K = p.K;
  a.N = p.N;
  a.ntiles = p.ntiles;
  a.kst = p.K / 32;
  a.W = p.W;
  a.P = p.P;
  a.tg = p.tg;
  a.ldo = c.ldo;
  a.epi = c.epi;
  a.layer = c.layer;
  a.start_pos = c.start_pos;
  a.n_q_heads = c.n_q_heads;
  a.eps = c.eps;
  a.row_tiles = row_tiles;
  a.act_tiles = c.act_tiles;
  a.gate = c.gate;
  if (c.gate != nullptr && row_tiles >= kWideMinRowTiles) return hipErrorInvalidValue;  // the wide kernel has no gate
  if (gemm_takes_wide(p, row_tiles, c.ssq_in != nullptr, c.wide_mode, n_cu, c.wide_ws ? c.wide_ws_bytes : 0))
    return launch_gemm_wide(c, a, st);
  if (c.m > kMaxPassRows) return hipErrorInvalidValue;
  const size_t lds = gemm_lds_floats(p.tg, p.W, 1, 1) * sizeof(float);
  const bool timed = c.ev_start != nullptr && c.ev_stop != nullptr;
  auto launch = [&](auto kernel) {
    if (timed)
      hipExtLaunchKernelGGL(kernel, dim3(p.grid), dim3(p.W * 64), (uint32_t)lds, st, c.ev_start, c.ev_stop, 0, a);
    else
      kernel<<<p.grid, p.W * 64, lds, st>>>(a);
  };
  // Few waves and narrow models (K = 2048: 4 waves, 128 partial sums per row): the sums of squares of all rows in one go,
  // 2 loads a row.  With 2 rows a wave and 8 loads a row, rows 8 and up are a second go, a memory latency more in
  // front of everything (1B shape, 9 rows, this and the additions across lanes on the vector unit: QKV 9.3 -> 8.2 us, gate/up
  // 16.8 -> 16.0, head 25.4 -> 24.7), but for up to 8 rows four would only be more to add (5 rows: gate/up 15.0 -> 15.9).
  // Eight waves have all rows in one go as it is; half the loads: 8B QKV 14.9 -> 14.6, gate/up 40.5 -> 40.3.
  //
  // Two row tiles: with the additions across lanes through the LDS unit and all eight loads, slower as each is by itself, the two
  // workgroups that read a tile's weights finish sooner (shown by exchanging one thing at a time: of 32 rows behind 1531 at
  // the 8B shape 4380 us on the vector unit with 4 loads, 4362 by shuffles, 4340 by shuffles with 8; why they then share the L2s better
  // is not).  Vector unit / this, medians over six model handles: 17 rows behind 777 3932 / 3938, prompts of 24 and 33 tokens 3562 / 3550 and
  // 3719 / 3691, 29 rows behind 3000 4672 / 4641, 32 behind 1531 4371 / 4342.  From three row tiles on it turns (33 to 62 rows
  // 3880 / 3888, 3872 / 3882, 3892 / 3895, 4370 / 4374), one has nobody to share with (9 rows 3468 / 3474), and so do models with four waves or
  // with phases (17 and 32 rows: 1B 1005 / 1016 and 1139 / 1136, 13B 1601 / 1609 and 1787 / 1791).
  const bool shuf = p.P == 1 && p.W == 8 && row_tiles == 2;
  auto launch_norm = [&](auto nt, auto epi, auto p1) {
    constexpr bool NT = decltype(nt)::value, P1 = decltype(p1)::value;
    constexpr int EPI = decltype(epi)::value;
    if constexpr (P1) {
      if constexpr (!NT) {
        if (shuf) return launch(gemm_bf16_kernel<16, NT, EPI, true, false, 2, kSsqPerLane, true>);
      }
      if (p.W == 8) return launch(gemm_bf16_kernel<16, NT, EPI, true, false, 2, 4>);  // (K = 4096: at most 256 partial sums)
      if (p.W < 8 && c.ssq_parts <= 2 * 64) {
        if (c.m <= 2 * p.W) return launch(gemm_bf16_kernel<16, NT, EPI, true, false, 2, 2>);
        return launch(gemm_bf16_kernel<16, NT, EPI, true, false, 4, 2>);
      }
    }
    launch(gemm_bf16_kernel<16, NT, EPI, P1>);
  };
  auto launch_p = [&](auto nt, auto p1) {
    constexpr bool NT = decltype(nt)::value, P1 = decltype(p1)::value;
    using std::integral_constant;
    switch (c.epi) {
      case EPI_STORE: launch_norm(nt, integral_constant<int, EPI_STORE>{}, p1); break;
      case EPI_RESID: launch(gemm_bf16_kernel<16, NT, EPI_RESID, P1>); break;
      case EPI_SWIGLU: launch_norm(nt, integral_constant<int, EPI_SWIGLU>{}, p1); break;
      default: launch_norm(nt, integral_constant<int, EPI_QKV>{}, p1); break;
    }
  };
  // Down projections: several K slices per wave and a tile for every team.  Awaiting a slice's
  // activations by themselves then drains the weight stream once per tile, so the next slice's travel
  // with its weights instead.  9 rows: 27.1 -> 25.2 us at the 8B shape (117 MB, 4 slices), 14.5 -> 14.6
  // at the 1B shape (34 MB, 2 slices).  With two tiles per team (17 rows and
  // more at the 8B shape) the same took 43 us against 36: 21 registers spill.
  const bool single_tile = c.epi == EPI_RESID && p.tg == 1 && p.ntiles <= p.grid / row_tiles;
  auto launch_nt = [&](auto nt) {
    if (p.P == 1)
      launch_p(nt, std::true_type{});
    else if (single_tile)
      launch(gemm_bf16_kernel<16, decltype(nt)::value, EPI_RESID, false, true>);
    else
      launch_p(nt, std::false_type{});
  };
  if (c.epi < EPI_STORE || c.epi > EPI_QKV) return hipErrorInvalidValue;
  // the residual epilogue is the one without a fused norm in front of it (compile-time knowledge of the kernels)
  if ((c.ssq_in != nullptr) != (c.epi != EPI_RESID)) return hipErrorInvalidValue;
  if (c.ssq_in != nullptr && c.ssq_parts > 64 * (p.P == 1 && p.W == 8 && !shuf ? 4 : kSsqPerLane)) return hipErrorInvalidValue;
  if (row_tiles == 1)
    launch_nt(std::true_type{});
  else
    launch_nt(std::false_type{});
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// re-tiling of the caller's row-major weights
// ------------------------------------------------------------------------------------------------
__global__ void pack_bf16_kernel(PackSrc s, int n_src, int K, int mode, int pair_span, uint4* __restrict__ dst,
                                 int ntiles) {
  const int kst = K / 32;
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;  // (tile, kstep, lane)
  const size_t total = (size_t)ntiles * kst * 64;
  if (idx >= total) return;
  const int lane = (int)(idx & 63);
  const int ks = (int)((idx >> 6) % kst);
  const int t = (int)((idx >> 6) / kst);
  const int i = lane & 15, g = lane >> 4;
  long vr;  // row in the stacked sources
  if (mode == PACK_PLAIN) {
    vr = (long)t * 16 + i;
  } else {
    const int tpg = pair_span / 8;  // tiles per group of 2 * pair_span rows
    const long base = (long)(t / tpg) * 2 * pair_span + (long)(t % tpg) * 8;
    vr = i < 8 ? base + i : base + pair_span + (i - 8);
  }
  uint4 v = make_uint4(0, 0, 0, 0);
  for (int j = 0; j < n_src; ++j) {
    if (vr < s.rows[j]) {
      v = *(const uint4*)(s.src[j] + (size_t)vr * K + ks * 32 + g * 8);
      break;
    }
    vr -= s.rows[j];
  }
  dst[idx] = v;
}

hipError_t launch_pack_bf16(const PackSrc& s, int n_src, int K, int mode, int pair_span, void* dst, int ntiles,
                            hipStream_t st) {
  const size_t total = (size_t)ntiles * (K / 32) * 64;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  pack_bf16_kernel<<<blocks, 256, 0, st>>>(s, n_src, K, mode, pair_span, (uint4*)dst, ntiles);
  return hipGetLastError();
}

}  // namespace pipesd
