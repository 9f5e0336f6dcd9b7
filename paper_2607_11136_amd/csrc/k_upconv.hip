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
// Nine sums in place of sixteen.  Along one axis the four sums have rank
// three: with a, b, c the products of a source pixel with the taps {0},
// {1, 2} and {2}, output 2i is a(i-1) + b(i) and output 2i-1 is
// a(i-1) + b(i-1) - c(i-1) + c(i).  So k_upconv multiplies every source pixel
// with the nine weights (a, b, c) x (a, b, c) only, and forms the four outputs
// from the products of neighbouring pixels in fp32: first along the columns
// (the neighbour is the lane to the left), then along the rows.  The four
// corner taps are single bf16 weights (lo is zero), the other five are hi +
// lo: 14 C_in C_out multiply-adds per source pixel, against 32 for the four
// phases by themselves and 36 for the convolution over the upsampled image.
//
// Tiling: 4 R x 16 source pixels x 32 channels a tile (R = 4, 3 or 2), each
// of eight waves R x 16 pixels x 16 channels as 9 R accumulators of
// v_mfma_f32_16x16x32.  A tile's first row and column only supply the tile's
// second ones (15 x 15 pixels of 16 x 16 are its own), except at the image's
// edge.  What a CU holds is bound by its accumulators: a wave reads R + 14
// fragments for 14 R MFMAs, and a K step of 64 channels loads 8 R + 56 KB
// for 224 R x 32 cycles of them.
//
// Persistent workgroups, one per CU, walk the tiles.  A workgroup per tile
// spent 9.4 us of 17.9 on its start, first loads, accumulator clearing and
// stores (vae_video); the steps of consecutive tiles follow one another here,
// and a tile is stored during the next one's first panels.
//
// Rows of a stage are whole cache lines (64 channels); with 32 a CU received
// 34 KB/us against 40.  Loads more than one unit ahead gained nothing: the
// main loop keeps 90% of the MFMA rate at the clock the chip holds under it
// (1.8 GHz), and 4 us a tile are left for the epilogue.
//
// 8 x 240 x 360, 256 -> 256 channels: 2.50 -> 1.22 ms; 33 of 67 rows of 90,
// 512 -> 512: 86 -> 30 us (four phases as 256 x 256 implicit GEMM tiles
// before).
//
// Determinism: every product sums its channels in one order (64 at a time, the
// panels of prod_p in turn, 32 channels an MFMA), and every output is the same
// expression of its products, whatever rows a call covers and whichever R its
// size picks; so a stage computed in row bands equals the stage computed at
// once.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace xema {

namespace {

constexpr int UT = 16;                    // source columns of a tile
constexpr int UCH = 32;                   // output channels of a tile
constexpr int UBK = 64;                   // channels per K step
constexpr int UROWB = UBK * 2;            // bytes of one operand row in a stage (a whole cache line)
constexpr int UNWAVES = 8;
constexpr int UPROD = 14;                 // weight panels: 9 tap sums, 5 of them as hi and lo
constexpr int UHALF = UPROD / 2;          // panels of a unit (half a step)
constexpr int UW_BYTES = UHALF * UCH * UROWB;
constexpr int UXS = 2, UWS = 3;           // LDS stages: steps of x, units of weights
constexpr int UGROUP = 8;                 // pixel tiles walked before the next channels
constexpr int UWGS = 256;                 // workgroups, one per CU
constexpr int UAHEAD = 5, URING = UHALF;  // weight fragments read ahead, and their registers

// Weight panel q: the summed weights of phase prod_p and source offset prod_t
// (hi, or lo where prod_lo), which belong to tap sum prod_acc = 3 r + c.
__host__ __device__ constexpr int prod_p(int q) {
  constexpr int v[UPROD] = {0, 1, 2, 3, 0, 0, 0, 0, 0, 0, 2, 2, 1, 1};
  return v[q];
}
__host__ __device__ constexpr int prod_t(int q) {
  constexpr int v[UPROD] = {0, 1, 2, 3, 1, 1, 2, 2, 3, 3, 3, 3, 3, 3};
  return v[q];
}
__host__ __device__ constexpr int prod_lo(int q) { return q >= 4 && (q & 1); }
__host__ __device__ constexpr int prod_acc(int q) {
  constexpr int v[UPROD] = {0, 2, 6, 8, 1, 1, 3, 3, 4, 4, 7, 7, 5, 5};
  return v[q];
}

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

// the value of the lane before, within its 16 lanes (0 for their first lane)
__device__ __forceinline__ float from_left(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x111, 0xf, 0xf, true));
}

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

template <int R>
__global__ __launch_bounds__(UNWAVES * 64, 1) void k_upconv(UpconvParams p) {
  constexpr int TR = 4 * R;                // source rows of a tile, R per wave
  constexpr int USTORES = 2 * R;           // stores of a wave per tile
  constexpr int UX_BYTES = TR * UT * UROWB, UW_AT = UXS * UX_BYTES;   // x of one step; the weights' stages
  __shared__ __attribute__((aligned(1024))) uint8_t smem[UW_AT + UWS * UW_BYTES];

  const int ci = p.ci, co = p.co, W = p.w, H = p.h;
  const int KT = ci / UBK;
  const int row_end = p.row_begin + p.row_count;
  const int base = max(p.row_begin - 1, 0);
  const int tiles_r = (row_end - base + TR - 2) / (TR - 1), tiles_c = (W + UT - 2) / (UT - 1);
  const int tiles_p = p.n * tiles_r * tiles_c, tiles_o = co / UCH;
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
  const int half = wave & 1, rows0 = (wave >> 1) * R;        // this wave's 16 channels and R tile rows
  const int l16 = lane & 15, l4 = lane >> 4;

  const __amdgpu_buffer_rsrc_t rx = rsrc(p.x, (int64_t)p.n * H * W * ci * 2);
  const __amdgpu_buffer_rsrc_t rw = rsrc(p.wp, (int64_t)64 * ci * co);

  struct Tile { int frame, i0, j0, n0; };   // the first source pixel and channel of a tile
  const Divisor per_group(UGROUP * tiles_o), by_tail(max(tiles_p % UGROUP, 1)), by_c(tiles_c), by_r(tiles_r);
  auto tile_at = [&](int t) {
    const int group = per_group.of(t), first_p = group * UGROUP;
    const int in_group = t - group * per_group.d;
    const int tn = tiles_p - first_p >= UGROUP ? in_group / UGROUP : by_tail.of(in_group);
    const int tp = first_p + in_group - tn * min(tiles_p - first_p, UGROUP);
    const int tr = by_c.of(tp), frame = by_r.of(tr);
    return Tile{frame, base + (tr - frame * tiles_r) * (TR - 1), (tp - tr * tiles_c) * (UT - 1), tn * UCH};
  };

  // A 1 KiB wave load fills 8 operand rows of a stage, lane l row l / 8 at
  // physical slot l % 8; slot j of row r holds the row's 16 bytes j ^ ((r >> 1) & 7),
  // so it fetches those.  x: wave w fills half rows R w .. R w + R - 1 of the tile; a
  // pixel outside the image is an offset beyond the buffer, which reads zeros.
  // Weights: of a unit's 28 groups of 8 rows, wave w fills w, w + 8, w + 16 and,
  // below 4, w + 24.
  const int lrow = lane >> 3, lslot = (lane & 7) ^ (lane >> 4);   // (of an even group of rows; ^ 4 for an odd one)
  const uint32_t w_off = (uint32_t)((8 * (wave & 3) + lrow) * 16 * ci + (lslot ^ (4 * (wave & 1))) * 16);
  uint32_t w_panel[2][4];     // byte offset of each load's panel at channel 0, per unit
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int q = UHALF * (c >> 2) + min((wave >> 2) + 2 * (c & 3), UHALF - 1);
    uint32_t ps = 0, ts = 0, ls = 0;   // prod_p, prod_t and prod_lo at a run-time q
#pragma unroll
    for (int k = 0; k < UPROD; ++k) {
      ps |= (uint32_t)prod_p(k) << (2 * k);
      ts |= (uint32_t)prod_t(k) << (2 * k);
      ls |= (uint32_t)prod_lo(k) << k;
    }
    const int pp = (ps >> (2 * q)) & 3, tt = ((ts >> (2 * q)) & 3) + 4 * ((ls >> q) & 1);
    w_panel[c >> 2][c & 3] = (uint32_t)(((int64_t)pp * co * 8 + tt) * ci * 2);
  }
  // What is loaded next: x of step ld_kt of tile ld_tile, at x_off, and the
  // weights of the step before it, at ld_w (those of the step itself are at
  // then_w).  Past the last tile x reads zeros and the weights are some tile's.
  int ld_tile = tile, ld_kt = 0;
  uint32_t x_off[R], ld_w = 0, then_w = 0;
  auto aim = [&]() {
    const bool valid = ld_tile < last;
    const Tile t = tile_at(valid ? ld_tile : tile);
#pragma unroll
    for (int c = 0; c < R; ++c) {
      const int g = wave * R + c, i = t.i0 + (g >> 1), j = t.j0 + 8 * (g & 1) + lrow;
      const uint32_t off = (uint32_t)((((int64_t)t.frame * H + i) * W + j) * ci * 2 + (lslot ^ (4 * (g & 1))) * 16);
      x_off[c] = valid && i < H && j < W ? off : 0x80000000u;
    }
    then_w = (uint32_t)(t.n0 * 16 * ci);
  };
  auto next_step = [&]() {
    ld_w = then_w;
    then_w += UROWB;
    if (++ld_kt == KT) {
      ld_kt = 0;
      ld_tile += UWGS / 8;
      aim();
    }
  };
  auto issue_x = [&](uint8_t* st, int c) {
    load_lds16(rx, st + (wave * R + c) * 1024, x_off[c], (uint32_t)(ld_kt * UROWB));
  };
  auto issue_w = [&](uint8_t* st, int hh, int c) {
    if (c < 3 || wave < 4) load_lds16(rw, st + (wave + 8 * c) * 1024, w_off, w_panel[hh][c] + ld_w);
  };

  // fragments: lane l reads operand row l % 16 of its block, logical slot 4 kk + l / 16
  const int frag_off = l16 * UROWB + ((l4 ^ (l16 >> 1)) * 16);
  f32x4 acc[9][R];
  bf16x8 xf[2][R], wf[URING];
  auto read_x = [&](const uint8_t* st, int kk, int r) {
    return *reinterpret_cast<const bf16x8*>(st + (rows0 + r) * 16 * UROWB + (frag_off ^ (64 * kk)));
  };
  auto read_w = [&](const uint8_t* st, int kk, int k) {
    return *reinterpret_cast<const bf16x8*>(st + (2 * k + half) * 16 * UROWB + (frag_off ^ (64 * kk)));
  };
  auto load_bias = [&](int ch) { return *reinterpret_cast<const u32x2*>(p.bias + ch + 16 * half + 4 * l4); };

  // Waits until at most N of this wave's loads and stores are in flight, and
  // meets the other waves.
  auto meet = [&](auto n) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(vm_imm(decltype(n)::value));
    barrier();
  };

  // The tile before: its outputs, to be stored while the next tile's first
  // panels run.  What is not the tile's goes to an offset beyond the row's
  // buffer, so every wave issues all USTORES stores.
  u32x4 done[USTORES];     // output row 2 (i0 + rows0 + k) - u of its lanes' columns at 2 k + u
  uint32_t done_col = 0x80000000u;
  int done_i = 0;                     // the source row of the wave's first tile row
  const uint16_t* done_y = p.y;       // output row 2 done_i - 1 at the tile's first column and channel
  const int64_t y_row = (int64_t)2 * W * co;
  auto store = [&](int s) {
    const int k = s >> 1, u = s & 1;
    const int i = done_i + k, src = i - u;    // the source row of output row 2i - u
    const bool mine = (rows0 + k > 0 || i == 0) && src >= p.row_begin && src < row_end;
    __builtin_amdgcn_raw_buffer_store_b128(done[s], rsrc(done_y + (2 * k + 1 - u) * y_row, mine ? 0x7fffffff : 0),
                                           done_col, 0, 0);
  };

  // A step in two units of UHALF panels, each of two k-steps of 32 channels, R
  // MFMAs a panel, one per tile row.  When a unit starts, the next one has
  // landed, and x of the next step before the second unit; unit u + 2 then goes
  // to the stage of unit u - 1 and, from the second unit on, x of the step
  // after next to the stage of this step's x, which is in registers by then.
  // Weight fragments are read UAHEAD panels ahead, across units.  Steps run on
  // from one tile to the next.  A tile's first step starts the sums, that of
  // (1, 2) x (1, 2) with the bias; the stores of the tile before (`stores`) may
  // still be in flight then.
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
    auto unit = [&](auto hh) {
      constexpr int HH = decltype(hh)::value;
      const uint8_t* here = w_ring + ws * UW_BYTES;
      uint8_t* freed = w_ring + (ws == 0 ? UWS - 1 : ws - 1) * UW_BYTES;
      ws = ws + 1 == UWS ? 0 : ws + 1;
      const uint8_t* next = w_ring + ws * UW_BYTES;
#pragma unroll
      for (int m = 0; m < 2 * UHALF; ++m) {
        const int kk = m / UHALF, k = m % UHALF, q = HH * UHALF + k, a = m + UAHEAD;
        wf[a % URING] = a < 2 * UHALF ? read_w(here, a / UHALF, a % UHALF) : read_w(next, 0, a - 2 * UHALF);
        // x: the second half of this step's rows, then the first of the next step's
        const int xr = HH == 0 ? m - 1 : m - UHALF - 1;
        const bool rx4 = xr >= 0 && xr < R;
        if (rx4) xf[HH ^ 1][xr] = HH == 0 ? read_x(x_here, 1, xr) : read_x(x_next, 0, xr);
        if (m < 4) issue_w(freed, HH, m);
        if (HH == 1 && m >= 5 && m < 5 + R) issue_x(x_here, m - 5);
        const bool st = FIRST && HH == 0 && m >= 4 && m < 4 + USTORES;
        if (st) store(m - 4);
        const int s = prod_acc(q);
#pragma unroll
        for (int r = 0; r < R; ++r)
          acc[s][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              wf[m % URING], xf[kk][r],
              FIRST && kk == 0 && !prod_lo(q) ? (s == 4 ? bv : f32x4{0.f, 0.f, 0.f, 0.f}) : acc[s][r], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, R / 2, 0);  // MFMA
        if (rx4)
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // LDS reads
        else
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (st) __builtin_amdgcn_sched_group_barrier(0x040, 1, 0);  // store
        if (m < 3 || (HH == 1 && m >= 5 && m < 5 + R)) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // global->LDS load
        __builtin_amdgcn_sched_group_barrier(0x008, R - R / 2, 0);
      }
    };
    // (what went out last may be in flight: x loads over the first unit, stores over the second)
    meet(std::integral_constant<int, R>());
    unit(std::integral_constant<int, 0>());
    meet(std::integral_constant<int, FIRST ? USTORES : 0>());
    unit(std::integral_constant<int, 1>());
    next_step();
  };

  aim();
#pragma unroll
  for (int c = 0; c < R; ++c) issue_x(smem, c);
  next_step();
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int c = 0; c < 4; ++c) issue_w(smem + UW_AT + u * UW_BYTES, u, c);
#pragma unroll
  for (int c = 0; c < R; ++c) issue_x(smem + UX_BYTES, c);
  next_step();
  u32x2 bias = load_bias(tile_at(tile).n0);
  meet(std::integral_constant<int, 3 + R>());    // (at least 3 + R loads went out after x and the first unit)
#pragma unroll
  for (int r = 0; r < R; ++r) xf[0][r] = read_x(smem, 0, r);
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

    // Epilogue.  acc[3 r + c][k][e] is the product of tap sum (r, c) at tile row
    // rows0 + k, column l16, channel n0 + 16 half + 4 l4 + e.  Along the columns
    // first: acc[3 r] becomes the row type's output at column 2j and acc[3 r + 1]
    // the one at 2j - 1.
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int k = 0; k < R; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a = acc[3 * r][k][e], b = acc[3 * r + 1][k][e], c = acc[3 * r + 2][k][e];
          float y0 = from_left(a) + b, y1 = from_left((a + b) - c) + c;
          asm volatile("" : "+v"(y0), "+v"(y1));   // (kept before the barrier, where the shifts fold into the additions)
          acc[3 * r][k][e] = y0;
          acc[3 * r + 1][k][e] = y1;
        }
    // then along the rows, the row above a wave's first one coming from the wave
    // before it, through the stage of the last unit
    static_assert(6 * 4096 <= UW_BYTES, "rows handed from wave to wave");
    meet(std::integral_constant<int, 63>());
    f32x4* xchg = reinterpret_cast<f32x4*>(smem + UW_AT + (ws == 0 ? UWS - 1 : ws - 1) * UW_BYTES) + lane;
    f32x4 up0[2], up1[2];    // of the row above: its tap row 0, and its rows 0 + (1, 2) - 2
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      up0[c] = up1[c] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (wave < 6) {
        xchg[(wave * 4 + c) * 64] = acc[c][R - 1];
        xchg[(wave * 4 + 2 + c) * 64] = (acc[c][R - 1] + acc[3 + c][R - 1]) - acc[6 + c][R - 1];
      }
    }
    meet(std::integral_constant<int, 63>());
    if (wave >= 2) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        up0[c] = xchg[((wave - 2) * 4 + c) * 64];
        up1[c] = xchg[((wave - 2) * 4 + 2 + c) * 64];
      }
    }
    // Lanes of 16-lane rows 2m and 2m + 1 swap halves, so that the first store
    // eight channels at column 2j and the second at 2j - 1.  The first column and
    // row of a tile are the halo of its neighbour, except at the image's edge.
    const int j = now.j0 + l16, odd = l4 & 1;
    const bool mine_col = odd ? l16 > 0 && j <= W : (l16 > 0 || j == 0) && j < W;
    done_col = mine_col ? (uint32_t)(((2 * l16 - odd) * co + 16 * half + 8 * (l4 >> 1)) * 2) : 0x80000000u;
    done_i = now.i0 + rows0;
    done_y = p.y + (((int64_t)now.frame * 2 * H + 2 * done_i - 1) * 2 * W + 2 * now.j0) * co + now.n0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        u32x2 o[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const f32x4 y = u ? up1[c] + acc[6 + c][k] : up0[c] + acc[3 + c][k];
          bf16x4 b;
#pragma unroll
          for (int e = 0; e < 4; ++e) b[e] = (bf16)y[e];
          o[c] = __builtin_bit_cast(u32x2, b);
        }
        const auto s0 = __builtin_amdgcn_permlane16_swap(o[0][0], o[1][0], false, false);
        const auto s1 = __builtin_amdgcn_permlane16_swap(o[0][1], o[1][1], false, false);
        done[2 * k + u] = u32x4{s0[0], s1[0], s0[1], s1[1]};
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        up0[c] = acc[c][k];
        up1[c] = (acc[c][k] + acc[3 + c][k]) - acc[6 + c][k];
      }
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

template <int R>
static hipError_t launch_rows(const UpconvParams& p, hipStream_t s) {
  const int base = p.row_begin > 0 ? p.row_begin - 1 : 0;
  const int64_t per_frame = (int64_t)((p.row_begin + p.row_count - base + 4 * R - 2) / (4 * R - 1)) *
                            ((p.w + UT - 2) / (UT - 1)) * (p.co / UCH);
  // (a launch's tiles are counted in 32 bits)
  const int step = (int)std::max<int64_t>(((int64_t)1 << 30) / per_frame, 1);
  for (int f = 0; f < p.n; f += step) {
    UpconvParams q = p;
    q.n = std::min(step, p.n - f);
    q.x = p.x + (int64_t)f * p.h * p.w * p.ci;
    q.y = p.y + (int64_t)f * 4 * p.h * p.w * p.co;
    const unsigned wgs = (unsigned)std::min<int64_t>(q.n * per_frame, UWGS);
    hipLaunchKernelGGL(k_upconv<R>, dim3(wgs), dim3(UNWAVES * 64), 0, s, q);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Tile rows by the rounds of tiles over the CUs times a tile's time, relative
// to R = 4: 0.8 at R = 3 and 0.62 at R = 2 (512 channels, one round: 22, 18.3
// and 15 us; many rounds: 0.78 and 0.57).  Measured at R = 4, 3, 2: 33 of 67
// rows of 90, 512 -> 512 channels 43.5, 36.6, 29.7 us; 40 x 100, 384 -> 256
// 22.5, 19.6, 24.0; 64 x 16 x 16, 256 -> 256 91, 75, 80; 90 x 120, 256 -> 256
// 28.2, 32.2, 31.9; 8 x 240 x 360, 256 -> 256 1224, 1312, 1518.
hipError_t launch_upconv(const UpconvParams& p, hipStream_t s) {
  const int base = p.row_begin > 0 ? p.row_begin - 1 : 0, rows = p.row_begin + p.row_count - base;
  const int64_t columns = (int64_t)p.n * ((p.w + UT - 2) / (UT - 1)) * (p.co / UCH);
  auto cost = [&](int R, int of_100) {
    const int64_t tiles = (rows + 4 * R - 2) / (4 * R - 1) * columns;
    return (tiles + UWGS - 1) / UWGS * of_100;
  };
  const int64_t c4 = cost(4, 100), c3 = cost(3, 80), c2 = cost(2, 62);
  if (c4 <= c3 && c4 <= c2) return launch_rows<4>(p, s);
  return c3 <= c2 ? launch_rows<3>(p, s) : launch_rows<2>(p, s);
}

}  // namespace xema
