// Which tile a call takes: the launchers' rules on sizes, free of device code
// so that they can be examined (and tested) on the host alone.
#pragma once

#include <cstdint>

namespace xema {

constexpr int RULE_CUS = 256;

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
