// Launch shapes of the bf16 products, and which of the two kernels a product takes: plain host arithmetic, free of
// HIP.
#pragma once

#include <stddef.h>

#include <algorithm>

namespace pipesd {

constexpr int kWideMinRowTiles = 3;

// ------------------------------------------------------------------------------------------------
// narrow kernel
// ------------------------------------------------------------------------------------------------
struct GemmPlan {  // launch shape of one GEMM
  int K, N, ntiles;
  int W, P, grid, tg;  // waves per workgroup, K phases per wave, workgroups, n-tiles per group
};

constexpr int kTmax16 = 7;  // n-tiles per group at W = 8 (the LDS reduce area stays under 64 KB)

// launch shape for the teams that `slots_cu` compute units hold at once (passes of more than one row tile: a part of the device,
// since every team's tiles are multiplied by a workgroup per row tile)
inline void shape_for(int N, int K, int slots_cu, GemmPlan& p) {
  p.K = K;
  p.N = N;
  p.ntiles = (N + 15) / 16;
  const int slices = K / 512;
  int W = 1;
  for (int cand = 8; cand >= 1; --cand)
    if (slices % cand == 0) { W = cand; break; }
  p.W = W;
  p.P = slices / W;
  const int slots = slots_cu * (8 / W > 0 ? 8 / W : 1);
  const int tmax = kTmax16 * 8 / W;
  int best_tg = 1;
  long best_cost = -1;
  for (int tg = 1; tg <= tmax; ++tg) {
    const int groups = (p.ntiles + tg - 1) / tg;
    const long rounds = (groups + slots - 1) / slots;
    const long cost = rounds * tg;
    if (best_cost < 0 || cost <= best_cost) { best_cost = cost; best_tg = tg; }
  }
  p.tg = best_tg;
  const int groups = (p.ntiles + p.tg - 1) / p.tg;
  p.grid = groups < slots ? groups : slots;
}

// Groups of workgroups are b, b + 8, ..: whole rounds of the 8 chiplets, and no more of them than the device holds at
// once (40 groups of 7 on 256 compute units, 36 rounded up, took 53 us for 8B QKV, 32 groups take 31; 96 rows of 8B gate/up in
// 48 groups of 6 185 us, in 40 102).
inline GemmPlan gemm_narrow_plan(int N, int K, int row_tiles, int n_cu) {
  GemmPlan p;
  shape_for(N, K, row_tiles == 1 ? n_cu : std::max(8, n_cu / row_tiles / 8 * 8), p);
  if (row_tiles > 1) p.grid = (p.grid + 7) / 8 * 8 * row_tiles;
  return p;
}

// About how long this kernel takes in groups of row_tiles workgroups: a start and an end, and what a compute unit
// reads of the weights, at 52 to 62 GB/s; phases cost another 15 %.  Within 15 % of the measured times of most products of the 1B,
// 8B and 13B shapes at 33 to 128 rows.  8B QKV, microseconds, narrow / wide with its rstd kernel: 48 rows 18.3 / 23.8, 64
// 20.1 / 26.0, 80 24.6 / 25.2, 112 30.7 / 28.7; 8B gate/up 48 rows 71 / 52; 1B gate/up 64 rows 26 / 28, 80 30 / 27.
// (Beyond 8 row tiles the wide kernel runs whatever this says: groups of 10 or 12 workgroups per stream
// took up to three times as long as groups of 8 or 16.)
inline double gemm_narrow_us(const GemmPlan& p, int row_tiles, int n_cu) {
  const int groups = (p.ntiles + p.tg - 1) / p.tg, streams = p.grid / row_tiles;  // (the grid of whole groups)
  const double mb = (double)((groups + streams - 1) / streams) * p.tg * p.K * 32e-6 * std::max(1.0, (double)p.grid / n_cu);
  const double mbs = row_tiles <= 3 ? 0.052 : row_tiles <= 5 ? 0.057 : 0.062;
  return (6.5 + mb / mbs) * (p.P > 1 ? 1.15 : 1.0);
}

// ------------------------------------------------------------------------------------------------
// wide kernel
// ------------------------------------------------------------------------------------------------
// the narrow kernel's split of K (W waves x P phases of 512 columns), which fixes the order of the sums
inline void wide_roles(int K, int& W, int& P) {
  W = 1;
  for (int cand = 8; cand >= 1; --cand)
    if ((K / 512) % cand == 0) { W = cand; break; }
  P = K / 512 / W;
}

struct WidePlan {
  int ct, rt;  // n-tiles per workgroup: 16 (2 x 4 waves of rt x 4 tiles) or 8 (4 x 2 waves); row tiles per wave
  bool whole;
  int block_tiles, nrb;
  double us;
};
constexpr size_t kWideSplitBytes = (size_t)128 << 20;  // the most that split products' running sums may take

// Shapes of the kernel, and what a workgroup takes (microseconds): `step` for a k-step, `tile` more for each of its 16 x 16
// output tiles, `fin` per tile behind the last one (the epilogue, where it walks all of K); `tbs`: the rate its weights come at
// from memory when nothing else holds it up (TB/s).
struct WideShape {
  int ct, rt;
  double step, tile, fin, tbs;
};
constexpr WideShape kWideShapes[] = {{16, 2, 0.35, 0.0014, 0.050, 6.2}, {16, 3, 0.44, 0.0010, 0.095, 6.3}, {16, 4, 0.49, 0.0012, 0.095, 4.9},
                                     {8, 1, 0.25, 0.0006, 0.0, 6.2},    {8, 2, 0.38, 0.0006, 0.060, 5.6},  {8, 3, 0.31, 0.0028, 0.075, 3.6}};

// Shape of a product by a model of its time.  A workgroup takes 1.7 us, its k-steps and its end, and 1.1 for every role
// whose total it keeps in memory; one workgroup runs per compute unit (a last round that is not full is up to 3 %
// shorter), of the smallest shape two, in 1.74 times the time of one; 3.7 lie around it all, and the second
// kernel of a split product takes 1.7 and its running sums at 2.1 TB/s.  So few rows take narrow tiles or a split of K, many
// rows 128 x 256 outputs per workgroup, and what decides in between is how full the last round of workgroups is; the end of
// large tiles, 10 us, is what a short walk (K of 512 to 1536) must not have twice.
//
// The figures are a fit to 25 000 timed products, two sessions: the four of 14 model shapes from 512 to 8192 columns, 33 to 2047
// rows, every shape, whole and split.  The shape they choose takes 0.5 % longer than the fastest one in the mean, 3 % in 19 of 20
// products and at most 31 % (512 columns, 2.5 us).  Fitted to a part of the 14 and tried on the rest it is 0.8 %, 5 % and 25 %.
// Before: a fit to the 1B, 8B and 13B shapes alone, without `fin`, 0.85 %, 5 % and 31 % over the 14 and up to 19 % slower than
// an earlier rule where walks are short.  Us, that rule / that fit / this one: 1024 columns, gate/up 2047 rows 66.4 / 78.8 / 66.4, QKV
// 1200 rows 27.6 / 28.5 / 27.6; 1536 gate/up 1000 rows 125 / 145 / 125; 2560 gate/up 640 rows 131 / 141 / 129, QKV 2047 rows 141 / 155 /
// 135.  Of the 1B, 8B and 13B widths no product is more than 1 % slower than by that fit, and calls of 33 and more rows are 0 to 1.8 % faster.
inline WidePlan wide_plan(int N, int K, int row_tiles, int n_cu, size_t ws_bytes) {
  int W, P;
  wide_roles(K, W, P);
  const int ntiles = (N + 15) / 16;
  WidePlan best{};
  for (const WideShape& sh : kWideShapes)
    for (const bool whole : {true, false}) {
      const int tiles = (sh.ct == 16 ? 2 : 4) * sh.rt;
      WidePlan p{sh.ct, sh.rt, whole, 0, (row_tiles + tiles - 1) / tiles, 0.0};
      p.block_tiles = (row_tiles + p.nrb - 1) / p.nrb;  // (spread evenly)
      p.nrb = (row_tiles + p.block_tiles - 1) / p.block_tiles;
      const size_t ws = (size_t)ntiles * row_tiles * 1024 * (whole ? (P > 1 ? 1 : 0) : W);
      if (ws > (whole ? ws_bytes : std::min(ws_bytes, kWideSplitBytes))) continue;
      const int wgs = (ntiles + sh.ct - 1) / sh.ct * p.nrb * (whole ? 1 : W), steps = 16 * P * (whole ? W : 1);
      const int out = sh.ct * p.block_tiles;
      const double one = 1.7 + steps * (sh.step + sh.tile * out) + (whole ? sh.fin * out + (P > 1 ? 1.1 * W : 0.0) : 0.0);
      double us;
      if (sh.ct == 8 && sh.rt == 1) {
        const int left = wgs % (2 * n_cu);
        us = one * (1.74 * (wgs / (2 * n_cu)) + (left == 0 ? 0.0 : left <= n_cu ? 1.0 : 1.74));
      } else {
        const int left = wgs % n_cu;
        us = one * (wgs / n_cu + (left == 0 ? 0.0 : 0.97 + 0.03 * left / n_cu));
      }
      us = 3.7 + std::max(us, (double)ntiles * 16 * K * 2e-6 / sh.tbs);
      if (!whole) us += 1.7 + (double)ws / 2.1e6;
      p.us = us;
      if (best.ct == 0 || us < best.us) best = p;
    }
  return best;
}

// Against the narrow kernel: the kernel that computes rstd in front of a product with a norm takes 2.7 more, and a split counts
// for 1.5 more than the fit says, since it is the one that cards differ in (8B O 96 rows, narrow 20.2, split 17.7 and 23.9).
// What the choice loses against the faster of both kernels with 0 / 1.5 / 3 there, in the mean over the products of 33 to 128 rows of
// the 14 model shapes: 0.72 / 0.52 / 0.60 % (of the 1B, 8B and 13B widths 0.62 / 0.33 / 0.38 %).
inline double gemm_wide_us(int N, int K, int row_tiles, bool norm, int n_cu, size_t ws_bytes) {
  const WidePlan p = wide_plan(N, K, row_tiles, n_cu, ws_bytes);
  return p.us + (norm ? 2.7 : 0.0) + (p.whole ? 0.0 : 1.5);
}

// mode: GemmCall::wide_mode
inline bool gemm_takes_wide(const GemmPlan& narrow, int row_tiles, bool norm, int mode, int n_cu, size_t ws_bytes) {
  if (row_tiles < kWideMinRowTiles || mode == 1) return false;
  if (mode == 2 || row_tiles > 8) return true;
  return gemm_wide_us(narrow.N, narrow.K, row_tiles, norm, n_cu, ws_bytes) < gemm_narrow_us(narrow, row_tiles, n_cu);
}

// largest workspace any product with N weight rows and K columns asks for at up to max_rows rows
inline size_t gemm_wide_workspace_bytes(int N, int K, int max_rows) {
  int W, P;
  wide_roles(K, W, P);
  const size_t tiles = (size_t)((N + 15) / 16) * ((max_rows + 15) / 16) * 1024;
  return std::max(P > 1 ? tiles : 0, std::min(tiles * W, kWideSplitBytes));
}

}  // namespace pipesd
