// Which tile a call takes: the launchers' rules on sizes, free of device code
// so that they can be examined (and tested) on the host alone.
#pragma once

#include <algorithm>
#include <cstdint>
#include <utility>
#include <vector>

namespace xema {

constexpr int RULE_CUS = 256;

// ---------------------------------------------------------------------------
// GEMM
// ---------------------------------------------------------------------------

// Completion time of n_big full tiles, then n_small half-height tiles costing
// `half` of a full one, dealt in order to the first free of the CUs (tiles
// freed at the same time form one group).
inline double tile_makespan(int64_t n_big, int64_t n_small, double half) {
  constexpr int64_t CUS = RULE_CUS;
  const int64_t rounds = n_big / CUS, extra = n_big % CUS;
  std::vector<std::pair<double, int64_t>> free_at;  // (time, CUs)
  if (CUS - extra) free_at.push_back({(double)rounds, CUS - extra});
  if (extra) free_at.push_back({(double)rounds + 1.0, extra});
  double end = free_at.back().first;
  if (n_big == 0) end = 0.0;
  while (n_small > 0) {
    size_t i = 0;
    for (size_t j = 1; j < free_at.size(); ++j)
      if (free_at[j].first < free_at[i].first) i = j;
    const double t = free_at[i].first;
    const int64_t k = std::min(free_at[i].second, n_small);
    n_small -= k;
    end = std::max(end, t + half);
    if (free_at[i].second == k) free_at.erase(free_at.begin() + i);
    else free_at[i].second -= k;
    bool merged = false;
    for (auto& g : free_at)
      if (g.first == t + half) { g.second += k; merged = true; }
    if (!merged) free_at.push_back({t + half, k});
  }
  return end;
}

// Rows [0, split) go to 256-row tiles, the rest to 128-row tiles: the split
// with the least modelled completion time.  A half-height tile costs 0.56 of a full
// one (8192 and 20480 rows of 12288 columns in either alone: 0.54 to 0.57, with the
// gated epilogue 0.52 to 0.60; any value from 0.53 to 0.62 gives the block's sizes the
// same times).  *rounds receives that time in full tiles.
inline int64_t gemm_row_split(int64_t M, int tiles_n, double* rounds) {
  constexpr double HALF = 0.56;
  const int64_t tm = (M + 255) / 256;
  int64_t best_split = M;
  double best = tile_makespan(tm * tiles_n, 0, HALF);
  for (int64_t t1 = tm - 1; t1 >= 0 && t1 >= tm - 16; --t1) {
    const int64_t rest = (M - t1 * 256 + 127) / 128;
    const double cost = tile_makespan(t1 * tiles_n, rest * tiles_n, HALF);
    if (cost < best - 1e-9) { best = cost; best_split = t1 * 256; }
  }
  *rounds = best;
  return best_split;
}

// The tiles of k_gemm_192 and k_gemm_ring, and last that of k_gemm, with the
// microseconds one 64-wide K step of a tile takes and what a tile costs beside its
// steps when every CU holds one (its pipeline's start and the latency of its
// epilogue; the time of the stores themselves is the same for all tiles).  A CU
// fetches about 55 GB/s from beyond its L2, so the small tiles cost their operand
// bytes and only the 256-row ones their MFMAs.
enum GemmTile { G256x192, G256x128, G128x192, G128x128, G128x96, G64x128, G64x64, GEMM_MAIN };
struct GemmCost { int rows, cols; double step_us, tile_us; };
constexpr GemmCost kGemmCost[] = {{256, 192, 1.14, 3},  {256, 128, 0.86, 3}, {128, 192, 0.76, 3}, {128, 128, 0.6, 2},
                                  {128, 96, 0.45, 1.5}, {64, 128, 0.33, 1},  {64, 64, 0.23, 1},  {256, 256, 1.44, 4}};

// The tile for an M x N problem of depth K: the fewest rounds over the CUs times a
// round's time; `split` is k_gemm's.  heads_dim: 64 or 128 for the QKV epilogue,
// which needs 64 columns a wave and, at 128, two waves a row.
//
// Over 950 problems (16 to 20480 rows, N of 256 to 12288, K of 64 to 12288, the three
// epilogues) the picked tile takes 0.5% more than the fastest one in the mean and
// 7% at most; with no fixed cost for the smaller tiles it was 3.8%, and up to 39% at
// K = 256.  k_gemm alone and the picked tile, us:
//   256 x 3072 x 12288    64 x 64    118 and 47
//   512 x 3072 x 3072     64 x 128    39 and 20
//   1000 x 3072 x 12288   128 x 96   123 and 94
//   6000 x 768 x 768      128 x 192   32 and 19
//   9216 x 768 x 768      256 x 128   33 and 25
//   2048 x 12288 x 3072   256 x 192  165 and 134
//   4000 x 3072 x 3072    256 x 192   80 and 74
//   20480 x 12288 x 256   256 x 256  211 (256 x 128: 258)
// At 2048 x 3072 x 3072 and 12288 128 x 192 tiles and half-height ones are within 4%
// alone; beside the attention of the next chunk the former are 1% ahead.
struct GemmPick { int tile; int64_t split; };
inline GemmPick gemm_pick(int64_t M, int N, int K, int heads_dim) {
  GemmPick pick{GEMM_MAIN, 0};
  double rounds;
  pick.split = gemm_row_split(M, N / 256, &rounds);
  const double steps = K / 64;
  const GemmCost& full = kGemmCost[GEMM_MAIN];
  double cost = rounds * (full.step_us * steps + full.tile_us);
  for (int t = 0; t < GEMM_MAIN; ++t) {
    const GemmCost& c = kGemmCost[t];
    if (N % c.cols) continue;
    if (heads_dim && c.cols != 128 && !(heads_dim == 64 && t == G64x64)) continue;
    const int64_t tiles = ((M + c.rows - 1) / c.rows) * (N / c.cols);
    const double us = (double)((tiles + RULE_CUS - 1) / RULE_CUS) * (c.step_us * steps + c.tile_us);
    if (us < cost - 1e-9) { cost = us; pick.tile = t; }
  }
  return pick;
}

// ---------------------------------------------------------------------------
// k_upconv.  A tile is RG R fragments of 16 corners (a corner: the four outputs
// between four source pixels) and 128 / RG channels.
// ---------------------------------------------------------------------------
enum UpconvShape { ROWS_SHAPE, COLUMNS_SHAPE, FLAT_SHAPE };
constexpr int UT = 16;                    // corners of a fragment
constexpr int UBK = 64;                   // channels per K step
constexpr int UNWAVES = 8;
constexpr int UUNITS = 4, UHALF = 7;      // units of a K step, weight panels of a unit
constexpr int UXS = 2, UWS = 3;           // LDS stages: steps of x, units of weights

struct UpconvSize { int n, h, w, ci, co, row_begin, row_count; };
struct UpconvTile { int rg, r; UpconvShape shape; double step_us, tile_us; };

// The 1 KiB loads that a stage of x holds.
constexpr int upconv_x_loads(int rg, int r, UpconvShape shape) {
  const int w_bytes = UWS * UHALF * 16 * (UNWAVES / rg) * UBK * 2;
  return shape == FLAT_SHAPE      ? (160 * 1024 - w_bytes) / UXS / 1024
         : shape == COLUMNS_SHAPE ? ((rg + 1) * (UT * r + 1) + 7) / 8
                                  : ((rg * r + 1) * (UT + 1) + 7) / 8;
}

// Rows of a frame in the row of all corners: the row past a frame's last one is
// the row before the next one's first, unless these are rows of the images.
constexpr int upconv_frame_rows(int h, int row_begin, int row_count) {
  return row_count + (row_begin == 0 && row_count == h ? 1 : 2);
}

// The tiles of the first n frames.
inline int64_t upconv_tiles(const UpconvSize& p, int64_t n, int rg, int r, UpconvShape shape) {
  const int64_t corners = UT * rg * r, frame = (int64_t)upconv_frame_rows(p.h, p.row_begin, p.row_count) * (p.w + 1);
  const int64_t pixels = shape == FLAT_SHAPE      ? (n * frame + corners - 1) / corners
                         : shape == COLUMNS_SHAPE ? n * (p.row_count / rg + 1) * (p.w / (UT * r) + 1)
                                                  : n * (p.row_count / (rg * r) + 1) * (p.w / UT + 1);
  return pixels * (p.co / (16 * UNWAVES / rg));
}

// Whether the tiles of 16 rg r corners in a row can be used: x of a step fits its
// stage, and a tile's outputs lie within 2^31 bytes.
inline bool upconv_flat_fits(const UpconvSize& p, int rg, int r) {
  const int64_t corners = UT * rg * r, frame = (int64_t)upconv_frame_rows(p.h, p.row_begin, p.row_count) * (p.w + 1);
  return corners + p.w + 2 <= 8 * upconv_x_loads(rg, r, FLAT_SHAPE) &&
         (corners / frame + 2) * 8 * p.h * p.w * p.co < ((int64_t)1 << 31);
}

// The tiles, with the microseconds of a K step of 64 channels and what a tile
// costs beside its steps, all CUs busy (8 x 240 x 360, 256 and 512 -> 256
// channels; FLAT 64 x 16 x 16, 256 -> 256).  ROWS tiles fetch least per corner but
// round a call's corner rows up to 16 or 12 and its columns to 16; COLUMNS round
// to 4 and 48, for bands of few rows; FLAT ones round nothing, but hold x of W + 2
// corners more, so they are for narrow images, and the small ones for small calls.
constexpr UpconvTile kUpconvTiles[] = {{4, 4, ROWS_SHAPE, 4.4, 2.4},    {4, 3, ROWS_SHAPE, 3.4, 2.2},
                                       {4, 3, COLUMNS_SHAPE, 3.4, 2.3}, {4, 3, FLAT_SHAPE, 3.4, 2.3},
                                       {8, 2, FLAT_SHAPE, 2.5, 1.6},    {8, 1, FLAT_SHAPE, 1.75, 1.3}};
constexpr int kNumUpconvTiles = (int)(sizeof(kUpconvTiles) / sizeof(kUpconvTiles[0]));

// The tile with the fewest rounds over the CUs times what one takes.  Over 60
// shapes (1 to 8 frames of 3 x 1000 to 540 x 960, whole and in bands) the picked tile
// was within 7% of the fastest of the six; in us, picked against always 4 x 4 ROWS:
// 64 x 16 x 16, 256 -> 256 channels 61 and 142; 33 of 67 rows of 90, 512 -> 512 49 and
// 73; one of 540 rows of 960, 2 frames, 128 -> 256 20 and 44.
inline int upconv_pick(const UpconvSize& p) {
  int best = 0;
  double cost = 0;
  for (int t = 0; t < kNumUpconvTiles; ++t) {
    const UpconvTile& c = kUpconvTiles[t];
    if (c.shape == FLAT_SHAPE && !upconv_flat_fits(p, c.rg, c.r)) continue;
    const int64_t rounds = (upconv_tiles(p, p.n, c.rg, c.r, c.shape) + RULE_CUS - 1) / RULE_CUS;
    const double us = (double)rounds * (p.ci / UBK * c.step_us + c.tile_us);
    if (t == 0 || us < cost) { best = t; cost = us; }
  }
  return best;
}

}  // namespace xema
