// The VAE decoder's upsampling stage, fused: nearest 2x upsampling followed
// by a 3x3 convolution (zero padding 1, bias), computed straight from the
// low-resolution input so the 4x larger upsampled image never exists.  The
// paper fuses the operators around VAE upsampling to cut its short-lived
// activation peak (Sec. 5.2, "Localized chunking and fusion"; Sec. 8, memory
// mitigation primitives).
//
// Weights.  Output pixel (2i + py, 2j + px) sees the upsampled rows
// 2i+py-1 .. 2i+py+1, which are the source rows i+py-1 and i+py (two of the
// three kernel rows fall on the same source row), and likewise for columns.
// So each of the four output phases (py, px) is a 2x2 convolution of the
// zero-padded input with weights summed over the kernel taps that land on the
// same source pixel:
//   source offset a = 0, 1 takes kernel rows {0} and {1, 2} when py = 0,
//   and {0, 1} and {2} when py = 1 (the same for columns with px).
// k_upconv_prep forms the summed weights once per layer as fp32 sums and
// keeps each as a pair of bf16 values, hi = the sum rounded to bf16 and lo =
// the remainder rounded to bf16, which together carry it to about 2^-17 of
// its size.
//
// Every summed weight is applied as it is (its lo is zero where one tap lands on
// the source pixel): 28 C_in C_out multiply-adds per source pixel, against 36 for
// the convolution over the upsampled image.  The sums have rank three along each
// axis, so nine of them would do (14 multiply-adds, 1.19 in place of 1.83 ms for
// 8 x 240 x 360, 256 -> 256 channels), but only with outputs formed as differences:
// w0 + w1 as w0 + (w1 + w2) - w2 carries the error of w1 + w2, and with row 2 of
// the kernel 2^12 times the others the last output row is off by 2.6e-3 of its
// size in place of 1e-7.
//
// Tiling.  The four outputs (2i - u, 2j - v), u, v = 0, 1, see the same four source
// pixels (i - 1 .. i, j - 1 .. j): a corner.  A wave holds R fragments of 16 corners
// by 16 channels as 4 R accumulators of v_mfma_f32_16x16x32, and reads 28 weight
// fragments and 2 R to 4 R of x per 32 channels for 28 R MFMAs.  Tiles are 4 R by
// 16, 4 by 16 R, or 16 R RG corners in a row (tile_rules.h has the six in use and
// the rule).  What bounds the large ones is MFMA issue at the clock the power
// limit leaves: a 64-channel step of 16 x 16 corners x 32 channels takes 4.4 us on
// all CUs (1700 TFLOP/s), and a tile 2.4 us besides; the small ones are bound by the
// fetch of weights (112 KB a step for 32 channels, at about 40 KB/us a CU).
//
// Persistent workgroups, one per CU, walk the tiles; the steps of consecutive
// tiles follow one another, and a tile is stored during the next one's first
// panels.  Rows of a stage are whole cache lines (64 channels).
//
// Against four 2x2 phase convolutions as 256 x 256 implicit GEMM tiles: 8 x 240 x
// 360, 256 -> 256 channels 2.57 -> 1.84 ms; 33 of 67 rows of 90, 512 -> 512 90 ->
// 48 us; 1 x 16 x 16, 512 -> 512 79 -> 17 us.
//
// Determinism: every output sums its products in one order (64 channels at a time,
// the panels of units 0 to 3 in turn, 32 channels an MFMA), whatever rows a call
// covers and whichever tile its size picks; so a stage computed in row bands
// equals the stage computed at once.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "tile_rules.h"

namespace xema {

namespace {

constexpr int UROWB = UBK * 2;            // bytes of one operand row in a stage (a whole cache line)
constexpr int UGROUP = 8;                 // pixel tiles walked before the next channels
constexpr int UWGS = 256;                 // workgroups, one per CU
constexpr int UAHEAD = 5, URING = UHALF;  // weight fragments read ahead, and their registers

// Weight panel k of unit u: the summed weights of phase panel_p and source
// offset panel_t (hi, or lo where panel_lo).  The single taps (p = t) have no
// lo.  The first two units hold source column 0, the others column 1, and the
// four phases' first panels come first.
__host__ __device__ constexpr int panel_p(int u, int k) {
  constexpr int v[UUNITS][UHALF] = {
      {0, 1, 2, 3, 0, 1, 2}, {3, 1, 2, 3, 0, 3, 1}, {0, 1, 2, 3, 0, 1, 2}, {3, 0, 2, 3, 0, 1, 2}};
  return v[u][k];
}
__host__ __device__ constexpr int panel_t(int u, int k) {
  constexpr int v[UUNITS][UHALF] = {
      {0, 0, 0, 0, 2, 2, 2}, {2, 0, 0, 0, 2, 2, 2}, {1, 1, 1, 1, 3, 3, 3}, {3, 1, 1, 1, 3, 3, 3}};
  return v[u][k];
}
__host__ __device__ constexpr int panel_lo(int u, int k) { return (u & 1) && k > 0; }
constexpr bool panels_complete() {        // hi of all (p, t), lo of all but p = t, each once
  for (int p = 0; p < 4; ++p)
    for (int t = 0; t < 4; ++t)
      for (int lo = 0; lo < 2; ++lo) {
        int n = 0;
        for (int u = 0; u < UUNITS; ++u)
          for (int k = 0; k < UHALF; ++k)
            n += panel_p(u, k) == p && panel_t(u, k) == t && panel_lo(u, k) == lo && (t & 1) == u / 2;
        if (n != (lo && p == t ? 0 : 1)) return false;
      }
  return true;
}
static_assert(panels_complete(), "every product once");
// A unit's panels run over both k-steps of 32 channels; the order of the two
// (first in halves 0 and 3) keeps each fragment of x in use for two half units.
__host__ __device__ constexpr int unit_kk(int u, int half) { return half ^ (u == 1 || u == 2); }

constexpr int vm_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// 16 bytes per lane from buffer offset voff + soff straight into LDS (the host
// pass cannot check this builtin with a run-time scalar offset)
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t r, uint8_t* dst, uint32_t voff, uint32_t soff) {
#if __HIP_DEVICE_COMPILE__
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)dst, 16, voff, soff, 0, 0);
#endif
}

// Workgroup barrier that keeps LDS accesses and MFMAs on their side.
__device__ __forceinline__ void barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Division of 0 <= t < 2^31 by a uniform d > 0: the high half of t times
// floor(2^32 / d) is the quotient or one less.
struct Divisor {
  int d;
  uint32_t m;
  __device__ explicit Divisor(int d_) : d(d_), m(d_ == 1 ? 0xffffffffu : (uint32_t)(0x100000000ull / (uint32_t)d_)) {}
  __device__ __forceinline__ int of(int t) const {
    const int q = (int)__umulhi((uint32_t)t, m);
    return q + (t - q * d >= d ? 1 : 0);
  }
};

}  // namespace

// The phase-summed weights: s = the sum of w[o][ky][kx][c] over the kernel
// taps (ky, kx) of phase p = 2 py + px that land on source offset t = 2 a +
// b, in fp32 in ascending (ky, kx); wp[p][o][t][c] = hi = bf16(s) and
// wp[p][o][4 + t][c] = bf16(s - hi) (s - hi is exact in fp32).  One thread
// per (p, o, t, c) writes both.
__global__ void k_upconv_prep(const uint16_t* __restrict__ w, int ci, int co, uint16_t* __restrict__ wp) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)16 * co * ci;
  if (idx >= total) return;
  const int c = (int)(idx % ci);
  const int t = (int)((idx / ci) % 4);
  const int o = (int)((idx / ((int64_t)4 * ci)) % co);
  const int p = (int)(idx / ((int64_t)4 * ci * co));
  const int py = p >> 1, px = p & 1, a = t >> 1, b = t & 1;
  // kernel rows landing on source offset a: py = 0: {0} | {1, 2}; py = 1: {0, 1} | {2}
  const int r0 = (py == 0) ? (a == 0 ? 0 : 1) : (a == 0 ? 0 : 2);
  const int r1 = (py == 0) ? (a == 0 ? 0 : 2) : (a == 0 ? 1 : 2);
  const int c0 = (px == 0) ? (b == 0 ? 0 : 1) : (b == 0 ? 0 : 2);
  const int c1 = (px == 0) ? (b == 0 ? 0 : 2) : (b == 0 ? 1 : 2);
  float s = 0.f;
  for (int ky = r0; ky <= r1; ++ky)
    for (int kx = c0; kx <= c1; ++kx) s += bf16_bits_to_f32(w[(((int64_t)o * 3 + ky) * 3 + kx) * ci + c]);
  const bf16 hi = (bf16)s;
  const bf16 lo = (bf16)(s - (float)hi);
  uint16_t* row = wp + (((int64_t)p * co + o) * 8) * ci;
  row[(int64_t)t * ci + c] = __builtin_bit_cast(uint16_t, hi);
  row[(int64_t)(4 + t) * ci + c] = __builtin_bit_cast(uint16_t, lo);
}

// RG groups of waves (4 or 8) with R fragments of 16 corners each, 8 / RG groups of
// 16 channels.  SHAPE of a tile: ROWS, RG R corner rows of 16 columns; COLUMNS, RG
// corner rows of 16 R columns; FLAT, 16 RG R corners in a row of all frames' corners.
template <int RG, int R, UpconvShape SHAPE>
__global__ __launch_bounds__(UNWAVES * 64, 1) void k_upconv(UpconvParams p) {
  constexpr bool FLAT = SHAPE == FLAT_SHAPE, WIDE = SHAPE == COLUMNS_SHAPE;
  constexpr int TR = RG * R, CG = UNWAVES / RG, UCH = 16 * CG;   // fragments and channels of a tile
  constexpr int USTORES = 2 * R;           // stores of a wave per tile
  constexpr int WL = UHALF * UCH / 8, UW_BYTES = WL * 1024;      // 1 KiB loads and bytes of a unit of weights
  constexpr int WLW = (WL + UNWAVES - 1) / UNWAVES;              // loads of a wave, at most
  constexpr int TROWS = WIDE ? RG : TR, TCOLS = WIDE ? UT * R : UT;   // corner rows and columns of a tile (but FLAT)
  constexpr int UXP = TCOLS + 1;             // pixels of a row of x in a stage
  constexpr int XL_MAX = upconv_x_loads(RG, R, SHAPE);           // loads of x a stage holds
  constexpr int XLW = (XL_MAX + UNWAVES - 1) / UNWAVES;          // loads of a wave, at most and at least
  constexpr int XLMIN = (FLAT ? UT * TR / 8 : XL_MAX) / UNWAVES;
  constexpr int UX_BYTES = XL_MAX * 1024, UW_AT = UXS * UX_BYTES;   // x of one step; the weights' stages
  constexpr bool SHARED = SHAPE == ROWS_SHAPE;   // a fragment's lower x is the next one's upper
  constexpr int NX = SHARED ? R + 1 : 2 * R;     // fragments of x of a column and k-step
  constexpr int XPS = (NX + 4) / 5;              // read a panel
  static_assert(WLW <= 4 && 5 + XLW <= 2 * UHALF && 4 + USTORES <= 2 * UHALF, "a unit's slots");
  static_assert(UW_AT + UWS * UW_BYTES <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[UW_AT + UWS * UW_BYTES];

  const int ci = p.ci, co = p.co, W = p.w, H = p.h;
  const int KT = ci / UBK;
  const int row_end = p.row_begin + p.row_count;
  // tiles of the row_count + 1 by W + 1 corners of a frame; FLAT: of the corners of all frames in a row
  const int tiles_r = p.row_count / TROWS + 1, tiles_c = W / TCOLS + 1, frame_rows = upconv_frame_rows(H, p.row_begin, p.row_count);
  const int tiles_p = FLAT ? (p.n * frame_rows * (W + 1) + UT * TR - 1) / (UT * TR) : p.n * tiles_r * tiles_c;
  const int tiles_o = co / UCH;
  const int total = tiles_p * tiles_o;
  // XCD-aware order: each XCD walks a contiguous range of tiles, pixel tiles
  // fastest in groups of UGROUP, so that the 32 tiles it runs at once share 8
  // pixel tiles and 4 channel tiles
  const int xcd = blockIdx.x & 7;
  const int per = total >> 3, rem = total & 7;
  const int last = (xcd + 1) * per + min(xcd + 1, rem);
  int tile = xcd * per + min(xcd, rem) + (int)(blockIdx.x >> 3);
  if (tile >= last) return;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cg = wave % CG, rows0 = (wave / CG) * R;         // this wave's 16 channels and R fragments
  const int l16 = lane & 15, l4 = lane >> 4;

  const __amdgpu_buffer_rsrc_t rx = rsrc(p.x, (int64_t)p.n * H * W * ci * 2);
  const __amdgpu_buffer_rsrc_t rw = rsrc(p.wp, (int64_t)64 * ci * co);

  struct Tile { int frame, i0, j0, n0; };   // the first corner (FLAT: i0, counted over all frames) and channel of a tile
  const Divisor per_group(UGROUP * tiles_o), by_tail(max(tiles_p % UGROUP, 1));
  const Divisor by_c(FLAT ? W + 1 : tiles_c), by_r(FLAT ? frame_rows : tiles_r);
  auto tile_at = [&](int t) {
    const int group = per_group.of(t), first_p = group * UGROUP;
    const int in_group = t - group * per_group.d;
    const int tn = tiles_p - first_p >= UGROUP ? in_group / UGROUP : by_tail.of(in_group);
    const int tp = first_p + in_group - tn * min(tiles_p - first_p, UGROUP);
    if (FLAT) return Tile{0, tp * (UT * TR), 0, tn * UCH};
    const int tr = by_c.of(tp), frame = by_r.of(tr);
    return Tile{frame, p.row_begin + (tr - frame * tiles_r) * TROWS, (tp - tr * tiles_c) * TCOLS, tn * UCH};
  };

  // A 1 KiB wave load fills 8 operand rows of a stage, lane l row l / 8 at
  // physical slot l % 8.  Weights: row 'panel UCH + channel' keeps its 16 bytes j
  // at slot j ^ ((row >> 1) & 7); of a unit's WL loads, wave w issues w, w + 8, ...
  // x: pixel (r, c) of the tile is row UXP r + c; FLAT: pixel r of those in a row from
  // the tile's first corner's upper left one on is row r (the images stand in that
  // row W + 1 apart with one column, and where it is outside the image one row, of
  // zeros between).  The swizzle goes by the row, with ROWS by the column, so that it is
  // the same for all fragments; any 16 pixels in a row of x lie in all banks once
  // (the LDS serves lanes of two slots together, so at an odd first pixel 2 of 16
  // meet: 3% of the LDS cycles of 8 x 240 x 360, 256 -> 256 channels).
  // A pixel outside the image is an offset beyond the buffer, which reads zeros.
  const int lrow = lane >> 3;
  const uint32_t w_off = (uint32_t)((8 * (wave % (UCH / 8)) + lrow) * 16 * ci +
                                    ((lane & 7) ^ (lane >> 4) ^ (4 * (wave & 1))) * 16);
  static_assert(UNWAVES % (UCH / 8) == 0, "a wave's loads are of the same channels");
  uint32_t w_panel[UUNITS][WLW];     // byte offset of each load's panel at channel 0
#pragma unroll
  for (int u = 0; u < UUNITS; ++u) {
    uint32_t ps = 0, ts = 0, ls = 0;   // panel_p, panel_t and panel_lo at a run-time k
#pragma unroll
    for (int k = 0; k < UHALF; ++k) {
      ps |= (uint32_t)panel_p(u, k) << (2 * k);
      ts |= (uint32_t)panel_t(u, k) << (2 * k);
      ls |= (uint32_t)panel_lo(u, k) << k;
    }
#pragma unroll
    for (int c = 0; c < WLW; ++c) {
      const int k = min((wave + UNWAVES * c) / (UCH / 8), UHALF - 1);
      const int pp = (ps >> (2 * k)) & 3, tt = ((ts >> (2 * k)) & 3) + 4 * ((ls >> k) & 1);
      w_panel[u][c] = (uint32_t)(((int64_t)pp * co * 8 + tt) * ci * 2);
    }
  }
  const int xl = FLAT ? (UT * TR + W + 2 + 7) / 8 : XL_MAX;   // loads of x
  int x_at[XLW];                     // the pixel of each: 64 r + c (FLAT: r)
#pragma unroll
  for (int c = 0; c < XLW; ++c) {
    const int row = (wave + UNWAVES * c) * 8 + lrow;
    x_at[c] = FLAT ? row : (row / UXP) * 64 + row % UXP;
  }
  // What is loaded next: x of step ld_kt of tile ld_tile, at x_off, and the
  // weights of the two steps before it, at w_now and w_next (those of the step
  // itself are at w_then).  Past the last tile x reads zeros and the weights are
  // some tile's.
  int ld_tile = tile, ld_kt = 0;
  uint32_t x_off[XLW], w_now = 0, w_next = 0, w_then = 0;
  auto aim = [&]() {
    const bool valid = ld_tile < last;
    const Tile t = tile_at(valid ? ld_tile : tile);
#pragma unroll
    for (int c = 0; c < XLW; ++c) {
      int frame = t.frame, i, j, sw;
      bool in = valid;
      if (FLAT) {
        const int at = t.i0 + x_at[c], row = by_c.of(at);
        frame = by_r.of(row);
        i = p.row_begin - 1 + row - frame * frame_rows;
        j = at - row * (W + 1) - 1;
        in = in && frame < p.n;
        sw = (x_at[c] >> 1) & 7;
      } else {
        const int r = x_at[c] >> 6, col = x_at[c] & 63;
        i = t.i0 - 1 + r;
        j = t.j0 - 1 + col;
        in = in && r <= TROWS;
        sw = ((SHARED ? col : r * UXP + col) >> 1) & 7;
      }
      const uint32_t off =
          (uint32_t)((frame * H + i) * W + j) * (uint32_t)(ci * 2) + (uint32_t)(((lane & 7) ^ sw) * 16);
      x_off[c] = in && (uint32_t)i < (uint32_t)H && (uint32_t)j < (uint32_t)W ? off : 0x80000000u;
    }
    w_then = (uint32_t)(t.n0 * 16 * ci);
  };
  auto next_step = [&]() {
    w_now = w_next;
    w_next = w_then;
    w_then += UROWB;
    if (++ld_kt == KT) {
      ld_kt = 0;
      ld_tile += UWGS / 8;
      aim();
    }
  };
  auto issue_x = [&](uint8_t* st, int c) {
    if (c < XLMIN || wave + UNWAVES * c < xl)
      load_lds16(rx, st + (wave + UNWAVES * c) * 1024, x_off[c], (uint32_t)(ld_kt * UROWB));
  };
  auto issue_w = [&](uint8_t* st, int u, int c, uint32_t at) {
    if (c < WL / UNWAVES || wave < WL % UNWAVES)
      load_lds16(rw, st + (wave + UNWAVES * c) * 1024, w_off, w_panel[u][c] + at);
  };

  // fragments: lane l reads operand row l % 16 of its block (x: the pixels from
  // column b of the tile on), logical slot 4 kk + l / 16
  const int w_frag = (cg * 16 + l16) * UROWB + ((l4 ^ (l16 >> 1)) * 16);
  int x_frag[2][2];                // source row a (ROWS: that of the next fragment), column b
  const int x_row = FLAT ? W + 1 : UXP;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int at = (FLAT ? rows0 * UT : (SHARED ? rows0 : wave / CG) * UXP) + l16 + a * x_row + b;
      x_frag[a][b] = at * UROWB + ((l4 ^ (((SHARED ? l16 + b : at) >> 1) & 7)) * 16);
    }
  f32x4 acc[4][R];                 // phase, fragment
  bf16x8 xf[2][NX], wf[URING];
  auto read_x = [&](const uint8_t* st, int b, int kk, int f) {
    return *reinterpret_cast<const bf16x8*>(st + (SHARED ? f * (UXP * UROWB) : f % R * (UT * UROWB)) +
                                            (x_frag[SHARED ? 0 : f / R][b] ^ (64 * kk)));
  };
  auto read_w = [&](const uint8_t* st, int kk, int k) {
    return *reinterpret_cast<const bf16x8*>(st + k * (UCH * UROWB) + (w_frag ^ (64 * kk)));
  };
  auto load_bias = [&](int ch) { return *reinterpret_cast<const u32x2*>(p.bias + ch + 16 * cg + 4 * l4); };

  // Waits until at most N of this wave's loads and stores are in flight, and
  // meets the other waves.
  auto meet = [&](auto n) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(vm_imm(decltype(n)::value));
    barrier();
  };

  // The tile before: its outputs, to be stored while the next tile's first
  // panels run.  What is outside the image or the band goes to an offset beyond
  // the row's buffer, so every wave issues all USTORES stores.
  u32x4 done[USTORES];     // output row 2i - u of its lanes' corners at 2 k + u
  constexpr int ND = FLAT ? USTORES : WIDE ? R : 1;   // offsets of a lane: by store, fragment or column
  uint32_t done_at[ND];
  int done_i = 0;                     // the wave's first corner row
  const uint16_t* done_y = p.y;       // output row 2 done_i - 1, column 2 j0 - 1, the tile's first channel (FLAT: its first frame)
  const int64_t y_row = (int64_t)2 * W * co;
#pragma unroll
  for (int k = 0; k < ND; ++k) done_at[k] = 0x80000000u;
  auto store = [&](int s) {
    const int k = s >> 1, u = s & 1;
    const int down = SHARED ? k : 0, src = done_i + down - u;    // the source row of output row 2i - u
    const bool mine = FLAT || (src >= p.row_begin && src < row_end);
    __builtin_amdgcn_raw_buffer_store_b128(done[s],
                                           rsrc(done_y + (FLAT ? 0 : (2 * down + 1 - u) * y_row), mine ? 0x7fffffff : 0),
                                           done_at[FLAT ? s : WIDE ? k : 0], 0, 0);
  };

  // A step in UUNITS units of UHALF panels, each over two k-steps of 32 channels, R
  // MFMAs a panel, one per corner row.  When a unit starts, the next one has
  // landed, and x of the next step before the last unit; unit u + 2 then goes to
  // the stage of unit u - 1 and, in the last unit, x of the step after next to
  // the stage of this step's x, which is in registers by then.  Weight fragments
  // are read UAHEAD panels ahead, across units, and those of x half a unit.
  // Steps run on from one tile to the next.  A tile's first step starts the sums
  // with the bias; the stores of the tile before may still be in flight then.
  int xs = 0, ws = 0;      // the stages of the step's x and the unit's weights
  auto step = [&](auto first, u32x2 bias) {
    constexpr bool FIRST = decltype(first)::value;
    f32x4 bv;
    bv[0] = __uint_as_float(bias[0] << 16);
    bv[1] = __uint_as_float(bias[0] & 0xffff0000u);
    bv[2] = __uint_as_float(bias[1] << 16);
    bv[3] = __uint_as_float(bias[1] & 0xffff0000u);
    uint8_t* x_here = smem + xs * UX_BYTES;
    xs ^= 1;
    const uint8_t* x_next = smem + xs * UX_BYTES;
    uint8_t* w_ring = smem + UW_AT;
    auto unit = [&](auto uu) {
      constexpr int U = decltype(uu)::value, NU = (U + 1) % UUNITS;
      const uint8_t* here = w_ring + ws * UW_BYTES;
      uint8_t* freed = w_ring + (ws == 0 ? UWS - 1 : ws - 1) * UW_BYTES;
      ws = ws + 1 == UWS ? 0 : ws + 1;
      const uint8_t* next = w_ring + ws * UW_BYTES;
#pragma unroll
      for (int m = 0; m < 2 * UHALF; ++m) {
        const int half = m / UHALF, k = m % UHALF, kk = unit_kk(U, half), a = m + UAHEAD;
        wf[a % URING] = a < 2 * UHALF ? read_w(here, unit_kk(U, a / UHALF), a % UHALF)
                                      : read_w(next, unit_kk(NU, 0), a - 2 * UHALF);
        // x: (column 0, k-step 1) in the first half unit, (1, 1) in the last of
        // unit 1, (1, 0) right after it, (0, 0) of the next step in the last of all
        const bool x_half = half == (U == 1 || U == 3);
        const int x0 = (m - half * UHALF - 1) * XPS, x1 = x0 + XPS < NX ? x0 + XPS : NX;
        const int nx = x_half && x0 >= 0 && x1 > x0 ? x1 - x0 : 0;
#pragma unroll
        for (int f = x0; f < x0 + nx; ++f) {
          if (U == 0) xf[1][f] = read_x(x_here, 0, 1, f);
          if (U == 1) xf[1][f] = read_x(x_here, 1, 1, f);
          if (U == 2) xf[0][f] = read_x(x_here, 1, 0, f);
          if (U == 3) xf[0][f] = read_x(x_next, 0, 0, f);
        }
        const bool lw = m < WLW, lx = U == 3 && m >= 5 && m < 5 + XLW;
        if (lw) issue_w(freed, (U + 2) % UUNITS, m, U < 2 ? w_now : w_next);
        if (lx) issue_x(x_here, m - 5);
        const bool st = FIRST && U == 0 && m >= 4 && m < 4 + USTORES;
        if (st) store(m - 4);
        const int pp = panel_p(U, k), ta = panel_t(U, k) >> 1;
#pragma unroll
        for (int r = 0; r < R; ++r)
          acc[pp][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[m % URING], xf[kk][SHARED ? r + ta : ta * R + r],
                                                               FIRST && U == 0 && m < 4 ? bv : acc[pp][r], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, R / 2, 0);  // MFMA
        if (nx == 2)
          __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);  // LDS reads
        else if (nx == 1)
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        else
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (st) __builtin_amdgcn_sched_group_barrier(0x040, 1, 0);  // store
        if ((lw && m < WL / UNWAVES) || (lx && m - 5 < XLMIN))
          __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // global->LDS load
        __builtin_amdgcn_sched_group_barrier(0x008, R - R / 2, 0);
      }
    };
    // (what went out last may be in flight: x loads over the first unit, stores over the second)
    meet(std::integral_constant<int, XLMIN>());
    unit(std::integral_constant<int, 0>());
    meet(std::integral_constant<int, FIRST ? USTORES : 0>());
    unit(std::integral_constant<int, 1>());
    meet(std::integral_constant<int, 0>());
    unit(std::integral_constant<int, 2>());
    meet(std::integral_constant<int, 0>());
    unit(std::integral_constant<int, 3>());
    next_step();
  };

  aim();
#pragma unroll
  for (int c = 0; c < XLW; ++c) issue_x(smem, c);
  next_step();
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int c = 0; c < WLW; ++c) issue_w(smem + UW_AT + u * UW_BYTES, u, c, w_next);
#pragma unroll
  for (int c = 0; c < XLW; ++c) issue_x(smem + UX_BYTES, c);
  next_step();
  u32x2 bias = load_bias(tile_at(tile).n0);
  meet(std::integral_constant<int, WL / UNWAVES + XLMIN>());    // (at least these went out after x and the first unit)
#pragma unroll
  for (int f = 0; f < NX; ++f) xf[0][f] = read_x(smem, 0, 0, f);
#pragma unroll
  for (int k = 0; k < UAHEAD; ++k) wf[k] = read_w(smem + UW_AT, 0, k);
#pragma unroll
  for (int k = 0; k < USTORES; ++k) done[k] = u32x4{0, 0, 0, 0};
  while (true) {
    step(std::true_type(), bias);
    for (int kt = 1; kt < KT; ++kt) step(std::false_type(), bias);
    const Tile now = tile_at(tile);
    tile += UWGS / 8;
    bias = load_bias(tile_at(min(tile, last - 1)).n0);

    // Epilogue.  acc[2 u + v][k][e] is output (2i - u, 2j - v) of corner row i = i0 +
    // rows0 + k, j = j0 + l16, channel n0 + 16 cg + 4 l4 + e.  Lanes of 16-lane rows
    // 2m and 2m + 1 swap halves, so that the first store eight channels at column
    // 2j and the second at 2j - 1.
    const int odd = l4 & 1, ch = 16 * cg + 8 * (l4 >> 1);
    if (FLAT) {
      const int frame0 = by_r.of(by_c.of(now.i0));
      done_y = p.y + (int64_t)frame0 * 4 * H * W * co + now.n0;
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int at = now.i0 + (rows0 + k) * UT + l16, row = by_c.of(at), frame = by_r.of(row);
        const int i = p.row_begin + row - frame * frame_rows, j = at - row * (W + 1);
        const bool mine_col = frame < p.n && (odd ? j > 0 : j < W);
#pragma unroll
        for (int u = 0; u < 2; ++u)
          done_at[2 * k + u] =
              mine_col && i - u >= p.row_begin && i - u < row_end
                  ? (uint32_t)(((((frame - frame0) * H + i) * 2 - u) * 2 * W + 2 * j - odd) * co + ch) * 2u
                  : 0x80000000u;
      }
    } else {
#pragma unroll
      for (int k = 0; k < ND; ++k) {
        const int j = now.j0 + k * UT + l16;
        const bool mine_col = odd ? j > 0 && j <= W : j < W;
        done_at[k] = mine_col ? (uint32_t)(((2 * (k * UT + l16) + 1 - odd) * co + ch) * 2) : 0x80000000u;
      }
      done_i = now.i0 + (SHARED ? rows0 : wave / CG);
      done_y = p.y + (((int64_t)now.frame * 2 * H + 2 * done_i - 1) * 2 * W + 2 * now.j0 - 1) * co + now.n0;
    }
#pragma unroll
    for (int k = 0; k < R; ++k)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        u32x2 o[2];
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          bf16x4 b;
#pragma unroll
          for (int e = 0; e < 4; ++e) b[e] = (bf16)acc[2 * u + v][k][e];
          o[v] = __builtin_bit_cast(u32x2, b);
        }
        const auto s0 = __builtin_amdgcn_permlane16_swap(o[0][0], o[1][0], false, false);
        const auto s1 = __builtin_amdgcn_permlane16_swap(o[0][1], o[1][1], false, false);
        done[2 * k + u] = u32x4{s0[0], s1[0], s0[1], s1[1]};
      }
    if (tile >= last) break;
  }
#pragma unroll
  for (int k = 0; k < USTORES; ++k) store(k);
  // the loads past the last tile still write to LDS
  __builtin_amdgcn_s_waitcnt(vm_imm(0));
}

hipError_t launch_upconv_prep(const uint16_t* w, int ci, int co, uint16_t* wp, hipStream_t s) {
  const int64_t total = (int64_t)16 * co * ci;
  hipLaunchKernelGGL(k_upconv_prep, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, w, ci, co, wp);
  return hipGetLastError();
}

template <int RG, int R, UpconvShape SHAPE>
static hipError_t launch_tiles(const UpconvParams& p, const UpconvSize& size, hipStream_t s) {
  // (a launch's tiles are counted in 32 bits)
  const int step = (int)std::max<int64_t>(((int64_t)1 << 30) / upconv_tiles(size, 1, RG, R, SHAPE), 1);
  for (int f = 0; f < p.n; f += step) {
    UpconvParams q = p;
    q.n = std::min(step, p.n - f);
    q.x = p.x + (int64_t)f * p.h * p.w * p.ci;
    q.y = p.y + (int64_t)f * 4 * p.h * p.w * p.co;
    const unsigned wgs = (unsigned)std::min<int64_t>(upconv_tiles(size, q.n, RG, R, SHAPE), UWGS);
    hipLaunchKernelGGL((k_upconv<RG, R, SHAPE>), dim3(wgs), dim3(UNWAVES * 64), 0, s, q);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_upconv(const UpconvParams& p, hipStream_t s) {
  const UpconvSize size{p.n, p.h, p.w, p.ci, p.co, p.row_begin, p.row_count};
  static_assert(kNumUpconvTiles == 6, "a case for every tile");
#define XEMA_UPCONV_TILE(t) \
  case t: return launch_tiles<kUpconvTiles[t].rg, kUpconvTiles[t].r, kUpconvTiles[t].shape>(p, size, s)
  switch (upconv_pick(size)) {
    XEMA_UPCONV_TILE(0);
    XEMA_UPCONV_TILE(1);
    XEMA_UPCONV_TILE(2);
    XEMA_UPCONV_TILE(3);
    XEMA_UPCONV_TILE(4);
    XEMA_UPCONV_TILE(5);
    default: return hipErrorInvalidValue;
  }
#undef XEMA_UPCONV_TILE
}

}  // namespace xema
