// C = A B^T on gfx950 bf16/fp16 MFMA, with the block's fused epilogues
// (bias, bias + GELU-tanh, gated residual).  Steps a2, a5, a7, a8.
//
// Tiling: a BM x 256 output tile per workgroup (BM = 256 or 128), K in steps
// of 64.  Eight waves (two per SIMD) in a 2 x 4 grid each own a (BM/2) x 64
// sub-tile held as (BM/32) x 4 accumulators of v_mfma_f32_16x16x32.  Operand
// tiles go from HBM straight into LDS with buffer_load ... lds (no VGPR
// staging), in whole cache lines (128-byte row segments).  A has two stages
// and B three, all 160 KB of LDS, and fragments are read from LDS up to five
// panels of MFMAs ahead, across the step's one barrier (gemm_tile has the
// order).  The main loop is bound by MFMA issue at the clock that the power
// limit leaves: a 64-wide step of a 256 x 256 tile takes 1.49 us on all 256
// CUs (1440 TFLOP/s), against 1.7 us with 32x32x16 MFMAs, two stages of each
// operand and reads one k-step ahead.  With all CUs at it a tile takes 7.6 us
// besides with 16-bit stores, 10 with GELU and 30 with the gated residual
// (20480 x 12288 at K = 64 to 1024).  The video block's launches, kernel trace:
//   QKV (17776 x 9216 x 3072) 858 -> 856 us, out-projection 364 -> 334 us, MLP up
//   (12288 x 3072) 1144 -> 1083 us, MLP down 1248 -> 1080 us
// The buffer descriptor of each tile covers only that tile's rows, so rows
// past M read as zero.
//
// One launch covers the rows in two tile heights: the first rows in 256-row
// tiles, the rest in 128-row tiles dispatched last, which fill the CUs the
// last round of full tiles leaves idle.  The split comes from a model of the
// completion time (gemm_row_split in tile_rules.h; e.g. 17776 x 3072 is 840 tiles
// of 256 x 256, four rounds over 256 CUs with the last 28% full; 54 tile-rows of
// 256 and 31 of 128 finish in about 3.6 rounds).
//
// Problems that these tiles would not spread over the CUs (chunks of a few
// hundred to a few thousand tokens, narrow layers) take smaller or narrower
// tiles with a deeper LDS ring instead (k_gemm_ring; gemm_pick has the rule).
//
// LDS layout: a stage of either operand holds its rows' 64 elements (128
// bytes = eight 16-byte slots) each; slot j of row r is stored at slot
// j ^ ((r >> 1) & 7).  The LDS has 64 four-byte banks and serves a 16-byte
// read for 16 lanes per cycle; those 16 lanes read 16 consecutive rows at
// one logical slot, and the swizzle spreads them over all 64 banks.
//
// The MFMA takes the weight fragment as its A operand and the activation
// fragment as its B operand, so each lane ends up holding four consecutive
// output features of one token row, and four 16-lane rows 16 of them: epilogue
// loads and stores are 16 bytes a lane, 64 contiguous bytes a row.
//
// Workgroups are dispatched round-robin over the 8 XCDs; the tile order
// below gives each XCD a contiguous range of tiles, walked in groups of 4
// tile-rows (1-2% faster than 8 on the block's shapes), so tiles that share
// operand panels share an L2.
//
// Determinism: every output element is the sum over ascending K in the MFMAs'
// own order, the same whatever M, the tile, the row maps or the tile position
// are, and a 16x16x32 MFMA's bits are those of two 32x32x16 ones in turn (the
// tests compare the tiles); so chunked and unchunked calls, and all tiles,
// agree bit for bit.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "kernels.h"
#include "tile_rules.h"

namespace xema {

namespace {

template <typename T>
struct Mfma;
template <>
struct Mfma<bf16> {
  typedef bf16x8 frag;
  static __device__ __forceinline__ f32x16 run(frag a, frag b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ f32x4 run16(frag a, frag b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<f16> {
  typedef f16x8 frag;
  static __device__ __forceinline__ f32x16 run(frag a, frag b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ f32x4 run16(frag a, frag b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};

constexpr int BN = 256, BK = 64;
constexpr int KS = BK / 16;                // MFMA k-steps per stage
constexpr int ROWB = BK * 2;               // bytes of one operand row in a stage
constexpr int SLOTS = BK / 8;              // 16-byte slots per row
constexpr int RPL = 1024 / ROWB;           // rows filled by one 1 KiB wave load
constexpr int B_BYTES = BN * BK * 2;       // B bytes per stage
constexpr int GROUP_M = 4;
constexpr int NWAVES = 8;                  // 2 x 4 waves, two per SIMD
constexpr int RING_GROUP_ROWS = 512;       // rows walked before the next columns (k_gemm_ring)
// slot swizzle of a 128-byte row (two rows share a 256-byte bank line)
__host__ __device__ constexpr int row_swz(int r) { return (r >> 1) & 7; }
constexpr int BUF_FLAGS = 0x00020000;      // raw buffer, 32-bit dwords

// 16 bytes per lane from buffer offset voff + soff straight into LDS (one
// 1 KiB wave row at dst).  The host pass cannot check this builtin with a
// run-time scalar offset, so it sees an empty body.
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t r, uint8_t* dst, uint32_t voff,
                                           uint32_t soff) {
#if __HIP_DEVICE_COMPILE__
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)dst, 16, voff, soff, 0, 0);
#endif
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                           BUF_FLAGS);
}

// (every element is rounded from its fp32 value, in both tile heights alike)
template <typename CT>
__device__ __forceinline__ void store4(CT* p, const float v[4]) {
  typedef CT c4 __attribute__((ext_vector_type(4)));
  c4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = from_f32<CT>(sizeof(CT) == 2 ? as_rounded_f32(v[e]) : v[e]);
  *reinterpret_cast<c4*>(p) = o;
}

// Two 8-column groups of one row, held as halves by lanes l (columns 0..3 of
// each group) and l^32 (columns 4..7): the lanes swap one half each, then the
// low lane stores group 0 and the high lane group 1, 16 bytes apiece.  `g0`
// points at group 0; a and b are this lane's halves of groups 0 and 1.
template <typename CT>
__device__ __forceinline__ void store_group_pair(CT* g0, const CT __attribute__((ext_vector_type(4))) a,
                                                 const CT __attribute__((ext_vector_type(4))) b, int hi,
                                                 bool valid) {
  typedef CT c4 __attribute__((ext_vector_type(4)));
  typedef CT c8 __attribute__((ext_vector_type(8)));
  static_assert(sizeof(c4) == 8, "16-bit elements");
  const u32x2 send = __builtin_bit_cast(u32x2, hi ? a : b);
  const auto r0 = __builtin_amdgcn_permlane32_swap(send[0], send[0], false, false);
  const auto r1 = __builtin_amdgcn_permlane32_swap(send[1], send[1], false, false);
  u32x2 got;  // the other lane's half: r[0] is the low lane's value, r[1] the high lane's
  got[0] = hi ? r0[0] : r0[1];
  got[1] = hi ? r1[0] : r1[1];
  const c4 other = __builtin_bit_cast(c4, got);
  c8 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    o[e] = hi ? other[e] : a[e];
    o[4 + e] = hi ? b[e] : other[e];
  }
  if (valid) *reinterpret_cast<c8*>(g0 + 8 * hi) = o;
}

template <typename RT>
__device__ __forceinline__ void load4f(const RT* p, float v[4]);
template <>
__device__ __forceinline__ void load4f<float>(const float* p, float v[4]) {
  const f32x4 u = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = u[e];
}
template <>
__device__ __forceinline__ void load4f<uint16_t>(const uint16_t* p, float v[4]) {
  const u32x2 u = *reinterpret_cast<const u32x2*>(p);
  v[0] = __uint_as_float(u[0] << 16);
  v[1] = __uint_as_float(u[0] & 0xffff0000u);
  v[2] = __uint_as_float(u[1] << 16);
  v[3] = __uint_as_float(u[1] & 0xffff0000u);
}

// s_waitcnt immediate: vmcnt[3:0] in bits 3:0 and vmcnt[5:4] in bits 15:14,
// expcnt in bits 6:4 (7 = no wait), lgkmcnt in bits 11:8 (0 = wait for all).
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }

// sum of the values of lanes l and l^32 (both lanes get the same result)
__device__ __forceinline__ float pair_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// LDS bytes the QKV epilogue uses on a BM-row tile at head_dim HD: the
// [BM] int4 token positions, at HD = 128 the [NW][WR] partial sums of squares
// (NW waves of WR rows each), and the [BM][HD/2 + 2] float2 (cos, sin) rows.
constexpr int qkv_epi_lds_bytes(int BM, int HD, int NW = NWAVES, int WR = 0) {
  return BM * 16 + (HD == 128 ? NW * (WR ? WR : BM / 2) * 4 : 0) + BM * (HD / 2 + 2) * 8;
}

// Epilogue of the QKV GEMM (EPI_QKV_HEADS at head_dim 64, EPI_QKV_HEADS_128
// at 128): steps a2 and a3 fused.  256 divides D, so a tile's columns lie in
// one section (Q, K or V).  A wave's 64 columns are one head at HD = 64, and
// one half of a head at HD = 128 (dims 64 * half .., half = wn % 2; the other
// half is in wave wn ^ 1 of the same rows).  Lane (r32, hi) holds, for each
// of its rows, the wave's columns 32 j + 8 q + 4 hi + e (j < 2, q < 4,
// e < 4), the rest being in lane r32 + 32 (1 - hi).  Q and K: v = acc + bias,
// RMS over the HD dims (at HD = 128 the two waves of a head exchange their
// partial sums of squares through LDS and add them in the same order, so
// both scale by the same factor), times gamma, the 3D RoPE rotation of the
// pairs (2p, 2p+1) and, for Q, the softmax factor log2(e)/sqrt(d), then one
// fp16 rounding; stored to [B, H, Lp, HD].  V: rounded to fp16 and
// transposed through LDS into [B, H, HD, Lp], 8 tokens per 16-byte store.
// Rows are the tokens tok_begin + (m mod rows_per_batch) of batch row
// m / rows_per_batch; nothing is written for m >= m_end.
template <int MI, int NJ, int BM, int HD, int NW, int WR>
__device__ __forceinline__ void epilogue_qkv_heads(const GemmParams& p, const f32x16 (&acc)[MI][NJ],
                                                   int64_t m0, int64_t m_end, int n0, int wm, int wn,
                                                   int lane, int wave, uint8_t* smem,
                                                   const uint16_t* __restrict__ bias) {
  static_assert(NJ == 2, "64 columns per wave");
  static_assert(HD == 64 || HD == 128, "head dims");
  constexpr int HALVES = HD / 64;   // waves per head
  constexpr int NP = HD / 2;        // rotated pairs per head
  const QkRopeArgs& a = p.qk;
  const int r32 = lane & 31, hi = lane >> 5;
  const int D = a.heads * HD;
  const int sect = n0 / D;
  const int h = (n0 - sect * D) / HD + wn / HALVES;
  const int half = wn % HALVES;
  const int64_t rpb = p.c_map.rows_per_batch;
  const int64_t Lp = a.padded_len;
  const int col0 = n0 + wn * 64 + 4 * hi;
  float bv[NJ][4][4];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) load4f<uint16_t>(bias + col0 + j * 32 + 8 * q, bv[j][q]);

  bool bad = false;  // an fp16 result at or beyond the fp16 range
  if (sect < 2) {
    const uint16_t* gam = sect == 0 ? a.q_gamma : a.k_gamma;
    float g[NJ][4][4];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) load4f<uint16_t>(gam + half * 64 + 4 * hi + j * 32 + 8 * q, g[j][q]);
    const float f = sect == 0 ? a.q_scale : 1.0f;
    f16* dst = sect == 0 ? a.q : a.k;
    // (cos, sin) of the tile's BM tokens x NP pairs, shared by its heads:
    // [BM][NP] float2 rows padded by 16 bytes (conflict-free 16-byte reads by
    // 16 consecutive rows), after [BM] int4 (valid, t, y, w) per token and,
    // at HD = 128, the partial sums of squares.  Pair p of a head rotates on
    // axis 0, 1 or 2 when it falls in that axis' range of the cumulative
    // dims/2 (table: axis-major, then position).
    constexpr int CS_STRIDE = NP + 2;  // float2 per padded row
    constexpr int SS_BYTES = HALVES > 1 ? NW * WR * 4 : 0;
    static_assert(qkv_epi_lds_bytes(BM, HD, NW, WR) == BM * 16 + SS_BYTES + BM * CS_STRIDE * 8, "LDS plan");
    int4* pos_lds = reinterpret_cast<int4*>(smem);
    float* ss_lds = reinterpret_cast<float*>(smem + BM * 16);
    float2* cs_lds = reinterpret_cast<float2*>(smem + BM * 16 + SS_BYTES);
    __syncthreads();  // every wave is done reading the operand stages
    {
      const int gw = max(a.geom.grid[2], 1), hw = max(a.geom.grid[1] * a.geom.grid[2], 1);
      for (int t = (int)threadIdx.x; t < BM; t += NW * 64) {
        const int64_t m = m0 + t;
        const bool valid = m < m_end;
        const int64_t bb = valid ? m / rpb : 0;
        const int vi = a.tok_begin + (int)(valid ? m - bb * rpb : 0) - a.text_len;
        const bool vis = valid && vi >= 0;
        pos_lds[t] = make_int4(vis ? 1 : 0, vis ? vi / hw : 0, vis ? (vi % hw) / gw : 0,
                               vis ? vi % gw : 0);
      }
    }
    __syncthreads();
    {
      const int np0 = a.geom.dims[0] / 2, np1 = a.geom.dims[1] / 2, np2 = a.geom.dims[2] / 2;
      const int tb1 = a.geom.grid[0] * np0, tb2 = tb1 + a.geom.grid[1] * np1;
      for (int e = (int)threadIdx.x; e < BM * NP; e += NW * 64) {
        const int t = e / NP, pr = e % NP;
        const int4 ps = pos_lds[t];
        int idx = -1;
        if (pr < np0) idx = ps.y * np0 + pr;
        else if (pr < np0 + np1) idx = tb1 + ps.z * np1 + (pr - np0);
        else if (pr < np0 + np1 + np2) idx = tb2 + ps.w * np2 + (pr - np0 - np1);
        cs_lds[t * CS_STRIDE + pr] = (ps.x && idx >= 0) ? a.table[idx] : make_float2(1.f, 0.f);
      }
    }
    if constexpr (HALVES > 1) {
      // this wave's sum of squares over its 64 dims, per row
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        float ss = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float v = acc[i][j][4 * q + e] + bv[j][q][e];
              ss = fmaf(v, v, ss);
            }
        ss = pair_sum(ss);
        if (hi == 0) ss_lds[wave * WR + i * 32 + r32] = ss;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int64_t m = m0 + wm * WR + i * 32 + r32;
      const bool valid = m < m_end;
      const int64_t bb = valid ? m / rpb : 0;
      const int tok = a.tok_begin + (int)(valid ? m - bb * rpb : 0);
      float v[NJ][4][4];
      float ss = 0.f;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[j][q][e] = acc[i][j][4 * q + e] + bv[j][q][e];
            ss = fmaf(v[j][q][e], v[j][q][e], ss);
          }
      if constexpr (HALVES > 1) {
        // dims 0..63 (wave wave - half) plus dims 64..127, in that order
        const float* sp = ss_lds + (wave - half) * WR + i * 32 + r32;
        ss = sp[0] + sp[WR];
      } else {
        ss = pair_sum(ss);
      }
      // 1/sqrt(mean + eps) with the hardware reciprocal square root (1 ulp)
      const float r = __builtin_amdgcn_rsqf(ss * (1.0f / (float)HD) + a.qk_eps);
      const float2* csr = cs_lds + (wm * WR + i * 32 + r32) * CS_STRIDE + half * 32 + 2 * hi;
      f16* row = dst + (((int64_t)bb * a.heads + h) * Lp + tok) * HD + half * 64;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        f16x4 o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          // pairs 16 j + 4 q + 2 hi + (0, 1)
          const f32x4 cc = *reinterpret_cast<const f32x4*>(csr + 16 * j + 4 * q);
#pragma unroll
          for (int e2 = 0; e2 < 2; ++e2) {
            const float2 cs = make_float2(cc[2 * e2], cc[2 * e2 + 1]);
            const float u0 = v[j][q][2 * e2] * r * g[j][q][2 * e2];
            const float u1 = v[j][q][2 * e2 + 1] * r * g[j][q][2 * e2 + 1];
            const float y0 = as_rounded_f32(fmaf(u0, cs.x, -u1 * cs.y) * f);
            const float y1 = as_rounded_f32(fmaf(u0, cs.y, u1 * cs.x) * f);
            bad |= valid && (!fits_f16(y0) || !fits_f16(y1));
            o[q][2 * e2] = (f16)y0;
            o[q][2 * e2 + 1] = (f16)y1;
          }
        }
#pragma unroll
        for (int q = 0; q < 4; q += 2) store_group_pair<f16>(row + j * 32 + 8 * q, o[q], o[q + 1], hi, valid);
      }
    }
    raise_flag(p.status, bad);
    return;
  }

  // V: every wave has finished reading the operand stages before they hold
  // the transposed blocks (16 KiB per wave at BM = 256)
  constexpr int TPW = WR;     // tokens of this wave's block
  __syncthreads();
  f16* lds = reinterpret_cast<f16*>(smem) + wave * 64 * TPW;   // [64 dims][TPW tokens]
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const bool valid = m0 + wm * WR + i * 32 + r32 < m_end;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float y = as_rounded_f32(acc[i][j][4 * q + e] + bv[j][q][e]);
          bad |= valid && !fits_f16(y);
          lds[(32 * j + 8 * q + 4 * hi + e) * TPW + i * 32 + r32] = (f16)y;
        }
  }
  raise_flag(p.status, bad);
  __syncthreads();
  for (int it = lane; it < 64 * (TPW / 8); it += 64) {
    const int d = it / (TPW / 8), g8 = it % (TPW / 8);
    const int64_t mf = m0 + wm * TPW + g8 * 8;
    if (mf >= m_end) continue;
    const f16x8 vals = *reinterpret_cast<const f16x8*>(lds + d * TPW + g8 * 8);
    const int64_t bb = mf / rpb, ii = mf - bb * rpb;
    const int tok = a.tok_begin + (int)ii;
    f16* vrow = a.vt + (((int64_t)bb * a.heads + h) * HD + half * 64 + d) * Lp;
    if (mf + 8 <= m_end && ii + 8 <= rpb && (tok & 7) == 0) {
      *reinterpret_cast<f16x8*>(vrow + tok) = vals;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int64_t m = mf + e;
        if (m < m_end) {
          const int64_t b2 = m / rpb;
          a.vt[(((int64_t)b2 * a.heads + h) * HD + half * 64 + d) * Lp + a.tok_begin + (m - b2 * rpb)] =
              vals[e];
        }
      }
    }
  }
}

}  // namespace

// Epilogue of a BM-row tile of NW waves, each holding WR = 32 MI rows and 64
// columns: the QKV heads, or bias (+ GELU | gated residual) and the stores.
template <int EPI, typename CT, typename RT, int MI, int NJ, int BM, int NW, int WR>
__device__ __forceinline__ void store_tile(const GemmParams& p, const f32x16 (&acc)[MI][NJ], int64_t m0,
                                           int64_t m_end, int n0, int wm, int wn, int lane, int wave,
                                           uint8_t* smem_raw, const uint16_t* __restrict__ bias,
                                           CT* __restrict__ cout, const RT* __restrict__ resid,
                                           const float* __restrict__ gate) {
  constexpr int WN = 32 * NJ;
  const int r32 = lane & 31, hi = lane >> 5;
  if constexpr (EPI == EPI_QKV_HEADS || EPI == EPI_QKV_HEADS_128) {
    epilogue_qkv_heads<MI, NJ, BM, EPI == EPI_QKV_HEADS ? 64 : 128, NW, WR>(p, acc, m0, m_end, n0, wm, wn, lane, wave,
                                                                            smem_raw, bias);
    return;
  }

  // Epilogue.  acc[i][j][r] = C[m][n] with m = m0 + wm*WR + i*32 + r32 and
  // n = n0 + wn*64 + j*32 + 8*(r/4) + 4*hi + r%4.  Every input of a row group
  // is loaded before any of its stores (the pointers are restrict), so the
  // loads overlap instead of each paying a full memory latency.
  float bv[NJ][4][4];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      load4f<uint16_t>(bias + n0 + wn * WN + j * 32 + 8 * q + 4 * hi, bv[j][q]);
  const int64_t rpb = p.c_map.rows_per_batch;
  bool bad = false;  // an fp16 result at or beyond the fp16 range
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int64_t m = m0 + wm * WR + i * 32 + r32;
    if (m >= m_end) continue;
    const int64_t b = m / rpb;
    const int64_t within = m - b * rpb;
    const int64_t crow = b * p.c_map.batch_stride + p.c_map.row_offset + within;
    CT* crow_ptr = cout + crow * p.ldc;
    float v[NJ][4][4];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[j][q][e] = acc[i][j][4 * q + e] + bv[j][q][e];
    if (EPI == XEMA_EPI_GATED_RESIDUAL) {
      const int64_t rrow = b * p.resid_map.batch_stride + p.resid_map.row_offset + within;
      const RT* rrow_ptr = resid + rrow * p.ld_resid;
      const float* grow = gate + b * p.gate_stride +
                          (p.gate_sel.pos_offset + within < p.gate_sel.text_len ? p.gate_sel.text_delta : 0);
      float res[NJ][4][4];
      f32x4 g[NJ][4];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int n = n0 + wn * WN + j * 32 + 8 * q + 4 * hi;
          load4f<RT>(rrow_ptr + n, res[j][q]);
          g[j][q] = *reinterpret_cast<const f32x4*>(grow + n);
        }
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[j][q][e] = fmaf(g[j][q][e], v[j][q][e], res[j][q][e]);
    }
    if (EPI == XEMA_EPI_BIAS_GELU) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[j][q][e] = gelu_tanh(v[j][q][e]);
    }
    if constexpr (sizeof(CT) == 2) {
      typedef CT c4 __attribute__((ext_vector_type(4)));
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
          c4 a, b;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float y0 = as_rounded_f32(v[j][q][e]), y1 = as_rounded_f32(v[j][q + 1][e]);
            if constexpr (__is_same(CT, f16)) bad |= !fits_f16(y0) || !fits_f16(y1);
            a[e] = from_f32<CT>(y0);
            b[e] = from_f32<CT>(y1);
          }
          store_group_pair<CT>(crow_ptr + n0 + wn * WN + j * 32 + 8 * q, a, b, hi, true);
        }
    } else {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          store4<CT>(crow_ptr + n0 + wn * WN + j * 32 + 8 * q + 4 * hi, v[j][q]);
    }
  }
  raise_flag(p.status, bad);
}

// Two 16-column blocks of one row, of which a lane of 16-lane row l4 holds
// columns 4 l4 .. 4 l4 + 3 each (a, b): rows 2m and 2m + 1 swap halves, then
// the first stores 8 columns of block a and the second of block b, 16 bytes
// apiece.  `base` points at block a.
template <typename CT>
__device__ __forceinline__ void store_block_pair(CT* base, const CT __attribute__((ext_vector_type(4))) a,
                                                 const CT __attribute__((ext_vector_type(4))) b, int l4, bool valid) {
  typedef CT c4 __attribute__((ext_vector_type(4)));
  static_assert(sizeof(c4) == 8, "16-bit elements");
  const u32x2 ua = __builtin_bit_cast(u32x2, a), ub = __builtin_bit_cast(u32x2, b);
  const auto r0 = __builtin_amdgcn_permlane16_swap(ua[0], ub[0], false, false);
  const auto r1 = __builtin_amdgcn_permlane16_swap(ua[1], ub[1], false, false);
  const u32x4 o = {r0[0], r1[0], r0[1], r1[1]};
  if (valid) *reinterpret_cast<u32x4*>(base + 16 * (l4 & 1) + 8 * (l4 >> 1)) = o;
}

// LDS bytes of one wave's transposed V block in epilogue_qkv_heads16: 64 dims
// of TPW tokens, padded so that the four dims a store meets lie in other banks.
constexpr int v_row(int TPW) { return TPW + 8; }

// epilogue_qkv_heads for 16x16 blocks: lane (l16, l4) holds, for tokens
// 16 i + l16 of the wave, the columns 16 j + 4 l4 + e (j < 4, e < 4).  The same
// operations in the same order per output.
template <int MI, int BM, int HD>
__device__ __forceinline__ void epilogue_qkv_heads16(const GemmParams& p, const f32x4 (&acc)[MI][4], int64_t m0,
                                                     int64_t m_end, int n0, int wm, int wn, int lane, int wave,
                                                     uint8_t* smem, const uint16_t* __restrict__ bias) {
  static_assert(HD == 64 || HD == 128, "head dims");
  constexpr int NW = NWAVES, WR = 16 * MI;
  constexpr int HALVES = HD / 64;   // waves per head
  constexpr int NP = HD / 2;        // rotated pairs per head
  const QkRopeArgs& a = p.qk;
  const int l16 = lane & 15, l4 = lane >> 4;
  const int D = a.heads * HD;
  const int sect = n0 / D;
  const int h = (n0 - sect * D) / HD + wn / HALVES;
  const int half = wn % HALVES;
  const int64_t rpb = p.c_map.rows_per_batch;
  const int64_t Lp = a.padded_len;
  float bv[4][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) load4f<uint16_t>(bias + n0 + wn * 64 + 16 * j + 4 * l4, bv[j]);

  bool bad = false;  // an fp16 result at or beyond the fp16 range
  if (sect < 2) {
    const uint16_t* gam = sect == 0 ? a.q_gamma : a.k_gamma;
    float g[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) load4f<uint16_t>(gam + half * 64 + 16 * j + 4 * l4, g[j]);
    const float f = sect == 0 ? a.q_scale : 1.0f;
    f16* dst = sect == 0 ? a.q : a.k;
    constexpr int CS_STRIDE = NP + 2;  // float2 per padded row
    constexpr int SS_BYTES = HALVES > 1 ? NW * WR * 4 : 0;
    static_assert(qkv_epi_lds_bytes(BM, HD, NW, WR) == BM * 16 + SS_BYTES + BM * CS_STRIDE * 8, "LDS plan");
    int4* pos_lds = reinterpret_cast<int4*>(smem);
    float* ss_lds = reinterpret_cast<float*>(smem + BM * 16);
    float2* cs_lds = reinterpret_cast<float2*>(smem + BM * 16 + SS_BYTES);
    __syncthreads();  // every wave is done reading the operand stages
    {
      const int gw = max(a.geom.grid[2], 1), hw = max(a.geom.grid[1] * a.geom.grid[2], 1);
      for (int t = (int)threadIdx.x; t < BM; t += NW * 64) {
        const int64_t m = m0 + t;
        const bool valid = m < m_end;
        const int64_t bb = valid ? m / rpb : 0;
        const int vi = a.tok_begin + (int)(valid ? m - bb * rpb : 0) - a.text_len;
        const bool vis = valid && vi >= 0;
        pos_lds[t] = make_int4(vis ? 1 : 0, vis ? vi / hw : 0, vis ? (vi % hw) / gw : 0, vis ? vi % gw : 0);
      }
    }
    __syncthreads();
    {
      const int np0 = a.geom.dims[0] / 2, np1 = a.geom.dims[1] / 2, np2 = a.geom.dims[2] / 2;
      const int tb1 = a.geom.grid[0] * np0, tb2 = tb1 + a.geom.grid[1] * np1;
      for (int e = (int)threadIdx.x; e < BM * NP; e += NW * 64) {
        const int t = e / NP, pr = e % NP;
        const int4 ps = pos_lds[t];
        int idx = -1;
        if (pr < np0) idx = ps.y * np0 + pr;
        else if (pr < np0 + np1) idx = tb1 + ps.z * np1 + (pr - np0);
        else if (pr < np0 + np1 + np2) idx = tb2 + ps.w * np2 + (pr - np0 - np1);
        cs_lds[t * CS_STRIDE + pr] = (ps.x && idx >= 0) ? a.table[idx] : make_float2(1.f, 0.f);
      }
    }
    // The sums of squares over this wave's 64 dims, per token, in the order of
    // epilogue_qkv_heads: columns 0..3 and 8..11 of each 16 in one chain, the
    // others in a second, then both added.  The lanes of 16-lane rows l4 and l4 + 2
    // hold the parts of one chain for two tokens; they trade halves, so that the
    // first has the whole chain of token block i and the second that of i + 1.
    float ss[MI];
    static_assert(MI % 2 == 0, "token blocks in pairs");
#pragma unroll
    for (int i = 0; i < MI; i += 2) {
      float sq = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float v0[4], v1[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[i][j][e] + bv[j][e]),
                                                          __float_as_uint(acc[i + 1][j][e] + bv[j][e]), false, false);
          v0[e] = __uint_as_float(r[0]);
          v1[e] = __uint_as_float(r[1]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) sq = fmaf(v0[e], v0[e], sq);
#pragma unroll
        for (int e = 0; e < 4; ++e) sq = fmaf(v1[e], v1[e], sq);
      }
      const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(sq), __float_as_uint(sq), false, false);
      const uint32_t both = __float_as_uint(__uint_as_float(r16[0]) + __uint_as_float(r16[1]));
      const auto r32 = __builtin_amdgcn_permlane32_swap(both, both, false, false);
      ss[i] = __uint_as_float(r32[0]);
      ss[i + 1] = __uint_as_float(r32[1]);
      if (HALVES > 1 && l4 == 0) {
        ss_lds[wave * WR + i * 16 + l16] = ss[i];
        ss_lds[wave * WR + (i + 1) * 16 + l16] = ss[i + 1];
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int64_t m = m0 + wm * WR + i * 16 + l16;
      const bool valid = m < m_end;
      const int64_t bb = valid ? m / rpb : 0;
      const int tok = a.tok_begin + (int)(valid ? m - bb * rpb : 0);
      float sum = ss[i];
      if constexpr (HALVES > 1) {
        // dims 0..63 (wave wave - half) plus dims 64..127, in that order
        const float* sp = ss_lds + (wave - half) * WR + i * 16 + l16;
        sum = sp[0] + sp[WR];
      }
      // 1/sqrt(mean + eps) with the hardware reciprocal square root (1 ulp)
      const float r = __builtin_amdgcn_rsqf(sum * (1.0f / (float)HD) + a.qk_eps);
      const float2* csr = cs_lds + (wm * WR + i * 16 + l16) * CS_STRIDE + half * 32 + 2 * l4;
      f16* row = dst + (((int64_t)bb * a.heads + h) * Lp + tok) * HD + half * 64;
      f16x4 o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        // pairs 8 j + 2 l4 + (0, 1)
        const f32x4 cc = *reinterpret_cast<const f32x4*>(csr + 8 * j);
#pragma unroll
        for (int e2 = 0; e2 < 2; ++e2) {
          const float2 cs = make_float2(cc[2 * e2], cc[2 * e2 + 1]);
          const float u0 = (acc[i][j][2 * e2] + bv[j][2 * e2]) * r * g[j][2 * e2];
          const float u1 = (acc[i][j][2 * e2 + 1] + bv[j][2 * e2 + 1]) * r * g[j][2 * e2 + 1];
          const float y0 = as_rounded_f32(fmaf(u0, cs.x, -u1 * cs.y) * f);
          const float y1 = as_rounded_f32(fmaf(u0, cs.y, u1 * cs.x) * f);
          bad |= valid && (!fits_f16(y0) || !fits_f16(y1));
          o[j][2 * e2] = (f16)y0;
          o[j][2 * e2 + 1] = (f16)y1;
        }
      }
#pragma unroll
      for (int j = 0; j < 4; j += 2) store_block_pair<f16>(row + 16 * j, o[j], o[j + 1], l4, valid);
    }
    raise_flag(p.status, bad);
    return;
  }

  // V: every wave has finished reading the operand stages before they hold
  // the transposed blocks
  constexpr int TPW = WR, VR = v_row(TPW);     // tokens of this wave's block, LDS row
  __syncthreads();
  f16* lds = reinterpret_cast<f16*>(smem) + wave * 64 * VR;   // [64 dims][TPW tokens]
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const bool valid = m0 + wm * WR + i * 16 + l16 < m_end;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float y = as_rounded_f32(acc[i][j][e] + bv[j][e]);
        bad |= valid && !fits_f16(y);
        lds[(16 * j + 4 * l4 + e) * VR + i * 16 + l16] = (f16)y;
      }
  }
  raise_flag(p.status, bad);
  __syncthreads();
  for (int it = lane; it < 64 * (TPW / 8); it += 64) {
    const int d = it / (TPW / 8), g8 = it % (TPW / 8);
    const int64_t mf = m0 + wm * TPW + g8 * 8;
    if (mf >= m_end) continue;
    const f16x8 vals = *reinterpret_cast<const f16x8*>(lds + d * VR + g8 * 8);
    const int64_t bb = mf / rpb, ii = mf - bb * rpb;
    const int tok = a.tok_begin + (int)ii;
    f16* vrow = a.vt + (((int64_t)bb * a.heads + h) * HD + half * 64 + d) * Lp;
    if (mf + 8 <= m_end && ii + 8 <= rpb && (tok & 7) == 0) {
      *reinterpret_cast<f16x8*>(vrow + tok) = vals;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int64_t m = mf + e;
        if (m < m_end) {
          const int64_t b2 = m / rpb;
          a.vt[(((int64_t)b2 * a.heads + h) * HD + half * 64 + d) * Lp + a.tok_begin + (m - b2 * rpb)] = vals[e];
        }
      }
    }
  }
}

// store_tile for 16x16 blocks: acc[i][j][e] = C[m][n] with m = m0 + wm WR +
// 16 i + l16 and n = n0 + 16 NJ wn + 16 j + 4 l4 + e; a store covers 64 contiguous
// bytes of each of 16 rows.
template <int EPI, typename CT, typename RT, int MI, int NJ, int BM>
__device__ __forceinline__ void store_tile16(const GemmParams& p, const f32x4 (&acc)[MI][NJ], int64_t m0, int64_t m_end,
                                             int n0, int wm, int wn, int lane, int wave, uint8_t* smem_raw,
                                             const uint16_t* __restrict__ bias, CT* __restrict__ cout,
                                             const RT* __restrict__ resid, const float* __restrict__ gate) {
  constexpr int WR = 16 * MI;
  if constexpr (EPI == EPI_QKV_HEADS || EPI == EPI_QKV_HEADS_128) {
    epilogue_qkv_heads16<MI, BM, EPI == EPI_QKV_HEADS ? 64 : 128>(p, acc, m0, m_end, n0, wm, wn, lane, wave, smem_raw,
                                                                 bias);
    return;
  }
  const int l16 = lane & 15, l4 = lane >> 4;
  const int nw = n0 + wn * 16 * NJ;
  float bv[NJ][4];
#pragma unroll
  for (int j = 0; j < NJ; ++j) load4f<uint16_t>(bias + nw + 16 * j + 4 * l4, bv[j]);
  const int64_t rpb = p.c_map.rows_per_batch;
  bool bad = false;  // an fp16 result at or beyond the fp16 range
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int64_t m = m0 + wm * WR + i * 16 + l16;
    const bool valid = m < m_end;    // (every lane takes part in the swaps)
    const int64_t mv = valid ? m : m0;
    const int64_t b = mv / rpb;
    const int64_t within = mv - b * rpb;
    CT* crow_ptr = cout + (b * p.c_map.batch_stride + p.c_map.row_offset + within) * p.ldc;
    float v[NJ][4];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[j][e] = acc[i][j][e] + bv[j][e];
    if (EPI == XEMA_EPI_GATED_RESIDUAL) {
      const RT* rrow_ptr = resid + (b * p.resid_map.batch_stride + p.resid_map.row_offset + within) * p.ld_resid;
      const float* grow = gate + b * p.gate_stride +
                          (p.gate_sel.pos_offset + within < p.gate_sel.text_len ? p.gate_sel.text_delta : 0);
      float res[NJ][4];
      f32x4 g[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        load4f<RT>(rrow_ptr + nw + 16 * j + 4 * l4, res[j]);
        g[j] = *reinterpret_cast<const f32x4*>(grow + nw + 16 * j + 4 * l4);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[j][e] = fmaf(g[j][e], v[j][e], res[j][e]);
    }
    if (EPI == XEMA_EPI_BIAS_GELU) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[j][e] = gelu_tanh(v[j][e]);
    }
    if constexpr (sizeof(CT) == 2) {
      typedef CT c4 __attribute__((ext_vector_type(4)));
      c4 o[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float y = as_rounded_f32(v[j][e]);
          if constexpr (__is_same(CT, f16)) bad |= valid && !fits_f16(y);
          o[j][e] = from_f32<CT>(y);
        }
#pragma unroll
      for (int j = 0; j < NJ; j += 2) store_block_pair<CT>(crow_ptr + nw + 16 * j, o[j], o[j + 1], l4, valid);
    } else {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (valid) store4<CT>(crow_ptr + nw + 16 * j + 4 * l4, v[j]);
    }
  }
  raise_flag(p.status, bad);
}

// One BM x BN_ output tile, in WMW x 8 / WMW waves of 16 MI x 16 NJ.  EPI: XEMA_EPI_BIAS / XEMA_EPI_BIAS_GELU (CT =
// bf16 or f16) or XEMA_EPI_GATED_RESIDUAL (CT = float, RT = residual element
// type).  Rows [m_begin, m_end) in tiles of BM rows; wg numbers this tile
// among them; smem_raw holds two stages of A and three of B.
template <typename T, int EPI, typename CT, typename RT, int BM, int BN_ = BN, int WMW = 2>
__device__ __forceinline__ void gemm_tile(const GemmParams& p, int64_t m_begin, int64_t m_end, int wg,
                                          uint8_t* smem_raw, const uint16_t* __restrict__ bias,
                                          CT* __restrict__ cout, const RT* __restrict__ resid,
                                          const float* __restrict__ gate) {
  static_assert(BM == 256 || BM == 128, "tile heights");
  constexpr int WNW = NWAVES / WMW, WR = BM / WMW, WCOLS = BN_ / WNW;
  constexpr int MI = WR / 16, NJ = WCOLS / 16;        // 16-row and 16-column blocks per wave
  constexpr int A_BYTES = BM * ROWB, B_BYTES = BN_ * ROWB;
  constexpr int A_LOADS = BM / NWAVES / RPL, B_LOADS = BN_ / NWAVES / RPL;  // 1 KiB loads per wave per step
  static_assert(A_LOADS * NWAVES * RPL == BM && B_LOADS * NWAVES * RPL == BN_ && NJ % 2 == 0, "load split");
  typedef typename Mfma<T>::frag frag;

  const int K = p.K;
  const int KT = K / BK;
  const int tiles_m = (int)((m_end - m_begin + BM - 1) / BM);
  const int tiles_n = p.N / BN_;
  const int total = tiles_m * tiles_n;
  // XCD-aware tile order (see the file comment)
  const int xcd = wg & 7, slot = wg >> 3;
  const int per = total >> 3, rem = total & 7;
  const int t = xcd * per + min(xcd, rem) + slot;
  const int group = t / (GROUP_M * tiles_n);
  const int first_m = group * GROUP_M;
  const int gsize = min(tiles_m - first_m, GROUP_M);
  const int in_group = t - group * GROUP_M * tiles_n;
  const int tm = first_m + in_group % gsize;
  const int tn = in_group / gsize;
  const int64_t m0 = m_begin + (int64_t)tm * BM;
  const int n0 = tn * BN_;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WNW, wn = wave % WNW;

  const T* A = reinterpret_cast<const T*>(p.a);
  const T* Bw = reinterpret_cast<const T*>(p.b);
  const int64_t bytes_a = min<int64_t>(BM, m_end - m0) * K * 2, bytes_b = (int64_t)BN_ * K * 2;

  // Direct-to-LDS load plan: a 1 KiB wave instruction fills RPL rows; wave w
  // fills A rows (BM/NWAVES) w .. and B rows (BN/NWAVES) w ..  Lane l writes
  // row l / SLOTS of its chunk at physical slot l % SLOTS, so it fetches the
  // logical slot that the row's swizzle maps there.  The row offset is the
  // VGPR operand, which the buffer range check covers: a row past M is out of
  // range whatever the K offset and reads zero, and a row inside stays inside
  // (row K + slot + k < (row + 1) K elements).
  uint32_t a_off[A_LOADS], b_off[B_LOADS];
#pragma unroll
  for (int c = 0; c < A_LOADS; ++c) {
    const int row = (wave * A_LOADS + c) * RPL + lane / SLOTS;
    a_off[c] = (uint32_t)((row * K + (((lane % SLOTS) ^ row_swz(row)) * 8)) * 2);
  }
#pragma unroll
  for (int c = 0; c < B_LOADS; ++c) {
    const int row = (wave * B_LOADS + c) * RPL + lane / SLOTS;
    b_off[c] = (uint32_t)((row * K + (((lane % SLOTS) ^ row_swz(row)) * 8)) * 2);
  }

  // The per-lane offsets above are loop-invariant: a step's K offset goes in
  // the instruction's scalar offset, so issuing a load costs no vector ALU
  // work.  A step past the last one (the pipeline runs ahead) goes to a stage
  // nobody reads, from a buffer of no bytes, which keeps the loop free of branches
  // and fetches nothing.  Tile offsets stay below 2^31, checked by the host.
  auto issue_a = [&](int kt, uint8_t* st, int c) {
    load_lds16(make_rsrc(A + m0 * K, kt < KT ? bytes_a : 0), st + (wave * A_LOADS + c) * 1024, a_off[c],
               (uint32_t)(kt * BK * 2));
  };
  auto issue_b = [&](int kt, uint8_t* st, int c) {
    load_lds16(make_rsrc(Bw + (int64_t)n0 * K, kt < KT ? bytes_b : 0), st + (wave * B_LOADS + c) * 1024, b_off[c],
               (uint32_t)(kt * BK * 2));
  };
  uint8_t* const b_ring = smem_raw + 2 * A_BYTES;

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // fragment addressing: lane l reads row l % 16 of a block, k-slot 4 kk + l / 16
  const int l16 = lane & 15, l4 = lane >> 4;
  const int frag_off = l16 * ROWB + ((l4 ^ (l16 >> 1)) * 16);
  const int a_frag = wm * WR * ROWB + frag_off, b_frag = wn * WCOLS * ROWB + frag_off;
  constexpr int AHEAD = MI == 8 ? 5 : 4, RING = 8;   // A fragments read ahead, and their registers
  frag fx[RING], fw[2][NJ];
  auto read_a = [&](const uint8_t* st, int kk, int i) {
    return *reinterpret_cast<const frag*>(st + (a_frag ^ (64 * kk)) + i * 16 * ROWB);
  };
  auto read_b = [&](const uint8_t* st, int kk, int j) {
    return *reinterpret_cast<const frag*>(st + (b_frag ^ (64 * kk)) + j * 16 * ROWB);
  };

  // Pipeline.  A step is 2 MI panels (a 16-row block of A at one of its two
  // k-steps) of NJ MFMAs.  A fragments are read AHEAD panels ahead and those
  // of B a k-step ahead, so that by panel MEET every wave has read all of step
  // kt, and from there on reads step kt+1.  At the barrier there, step kt+1 has
  // landed and A of step kt+2 goes to the stage of A freed; B has three stages,
  // so that of step kt+2 goes out at the start of step kt already.  With half
  // of the loads in flight for two steps, no panel waits for the fetch of 64 KB
  // within one step.
  constexpr int PANELS = 2 * MI, MEET = PANELS - AHEAD;
  constexpr int B1 = MI == 8 ? 3 : 0;        // the panel from which B of the second k-step is read, over four
  static_assert(B1 + 4 <= MEET && MEET + 4 <= PANELS && B_LOADS <= MEET, "step read before the barrier");
  static_assert(PANELS % RING == 0, "fragment registers");
  int bs = 0;                                // the stage of B of step kt
  auto step = [&](int kt) {
    uint8_t* a_here = smem_raw + (kt & 1) * A_BYTES;
    const uint8_t* a_next = smem_raw + ((kt & 1) ^ 1) * A_BYTES;
    const uint8_t* b_here = b_ring + bs * B_BYTES;
    bs = bs + 1 == 3 ? 0 : bs + 1;
    const uint8_t* b_next = b_ring + bs * B_BYTES;
    uint8_t* b_free = b_ring + (bs + 1 == 3 ? 0 : bs + 1) * B_BYTES;
#pragma unroll
    for (int m = 0; m < PANELS; ++m) {
      if (m == MEET) {
        // A and B of step kt+1 have landed; B of step kt+2 may be in flight
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(B_LOADS));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      const int kk = m / MI, i = m % MI, a = m + AHEAD;
      fx[a % RING] = a < PANELS ? read_a(a_here, a / MI, a % MI) : read_a(a_next, (a - PANELS) / MI, (a - PANELS) % MI);
      const bool rb1 = m >= B1 && m < B1 + 4, rb0 = m >= MEET && m < MEET + 4;
      const int nb = rb1 ? m - B1 : m - MEET, j0 = nb * NJ / 4, j1 = (nb + 1) * NJ / 4;
#pragma unroll
      for (int j = j0; j < j1; ++j) {
        if (rb1) fw[1][j] = read_b(b_here, 1, j);
        if (rb0) fw[0][j] = read_b(b_next, 0, j);
      }
      const bool lb = m < B_LOADS, la = m >= MEET && m < MEET + A_LOADS;
      if (lb) issue_b(kt + 2, b_free, m);
      if (la) issue_a(kt + 2, a_here, m - MEET);
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = Mfma<T>::run16(fw[kk][j], fx[m % RING], acc[i][j]);
      __builtin_amdgcn_sched_group_barrier(0x008, NJ / 2, 0);  // MFMA
      if ((rb1 || rb0) && j1 - j0 == 2)
        __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);  // LDS reads
      else if (rb1 || rb0)
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      else
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (lb || la) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // global->LDS load
      __builtin_amdgcn_sched_group_barrier(0x008, NJ / 2, 0);
    }
  };
#pragma unroll
  for (int c = 0; c < A_LOADS; ++c) issue_a(0, smem_raw, c);
#pragma unroll
  for (int c = 0; c < B_LOADS; ++c) issue_b(0, b_ring, c);
#pragma unroll
  for (int c = 0; c < B_LOADS; ++c) issue_b(1, b_ring + B_BYTES, c);
#pragma unroll
  for (int c = 0; c < A_LOADS; ++c) issue_a(1, smem_raw + A_BYTES, c);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(A_LOADS + B_LOADS));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < NJ; ++j) fw[0][j] = read_b(b_ring, 0, j);
#pragma unroll
  for (int m = 0; m < AHEAD; ++m) fx[m] = read_a(smem_raw, m / MI, m % MI);
  for (int kt = 0; kt < KT; ++kt) step(kt);
  // the loads of the last iterations still write to LDS: let them finish
  // before the epilogue or the workgroup's end
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));

  store_tile16<EPI, CT, RT, MI, NJ, BM>(p, acc, m0, m_end, n0, wm, wn, lane, wave, smem_raw, bias, cout, resid, gate);
}

// A BM x BN output tile, BN = 32 NJ WNW, for problems whose 256-column tiles
// would leave CUs idle: WMW x WNW waves of (BM/WMW) x 32 NJ, an NS-stage ring
// of 64-wide K steps, the same swizzled LDS rows, and the same MFMA sequence
// per output element as gemm_tile, so the results are its bits.
//
// What bounds the small tiles is the fetch: a CU gets about 55 GB/s of operand
// rows from beyond its L2 (93-128 GB/s from L2), whatever the number of loads
// in flight past about 48 KB, the access order within a row, or the number of
// waves; with the loads alone a 128 x 128 tile takes the same 0.54 us a step
// as the whole loop.  Hence tiles as large as still give each CU one, and a
// ring deep enough for that much in flight.
//
// Where the registers allow it, a wave reads all fragments of step kt+1 from
// LDS while the MFMAs of step kt run (64 x 64 tiles at K = 3072: 17 -> 13 us
// against one k-step ahead).  The barrier before them means that every wave
// holds step kt in registers, so its stage is free for step kt + NS, and that
// step kt+1 has landed, while the NS - 2 steps after it may be in flight.
template <typename T, int EPI, typename CT, typename RT, int BM, int WMW, int WNW, int NJ_, int NS_>
__device__ __forceinline__ void gemm_ring_tile(const GemmParams& p, int wg, uint8_t* smem_raw,
                                               const uint16_t* __restrict__ bias, CT* __restrict__ cout,
                                               const RT* __restrict__ resid, const float* __restrict__ gate) {
  constexpr int NW = WMW * WNW, WCOLS = 32 * NJ_, BN_ = WNW * WCOLS;
  constexpr int WR = BM / WMW;
  constexpr int MI = WR / 32;
  constexpr int A_BYTES = BM * ROWB, STAGE_BYTES = A_BYTES + BN_ * ROWB;
  constexpr int A_LOADS = BM / NW / RPL, B_LOADS = BN_ / NW / RPL;
  static_assert(MI * 32 * WMW == BM && A_LOADS * NW * RPL == BM && B_LOADS * NW * RPL == BN_, "tile split");
  static_assert(NS_ >= 2, "ring");
  constexpr int LPS = A_LOADS + B_LOADS;
  typedef typename Mfma<T>::frag frag;

  const int K = p.K;
  const int KT = K / BK;
  const int tiles_m = (int)((p.M + BM - 1) / BM);
  const int tiles_n = p.N / BN_;
  const int total = tiles_m * tiles_n;
  // each XCD walks a contiguous range of tiles, rows fastest in groups of
  // RING_GROUP_ROWS rows, so that a weight panel is read by few XCDs
  constexpr int GM = RING_GROUP_ROWS / BM;
  const int xcd = wg & 7, slot = wg >> 3;
  const int per = total >> 3, rem = total & 7;
  const int t = xcd * per + min(xcd, rem) + slot;
  const int group = t / (GM * tiles_n);
  const int first_m = group * GM;
  const int gsize = min(tiles_m - first_m, GM);
  const int in_group = t - group * GM * tiles_n;
  const int64_t m0 = (int64_t)(first_m + in_group % gsize) * BM;
  const int n0 = (in_group / gsize) * BN_;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WNW, wn = wave % WNW;

  const T* A = reinterpret_cast<const T*>(p.a);
  const T* Bw = reinterpret_cast<const T*>(p.b);
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(A + m0 * K, min<int64_t>(BM, p.M - m0) * K * 2);
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(Bw + (int64_t)n0 * K, (int64_t)BN_ * K * 2);

  uint32_t a_off[A_LOADS], b_off[B_LOADS];
#pragma unroll
  for (int c = 0; c < A_LOADS; ++c) {
    const int row = (wave * A_LOADS + c) * RPL + lane / SLOTS;
    a_off[c] = (uint32_t)((row * K + (((lane % SLOTS) ^ row_swz(row)) * 8)) * 2);
  }
#pragma unroll
  for (int c = 0; c < B_LOADS; ++c) {
    const int row = (wave * B_LOADS + c) * RPL + lane / SLOTS;
    b_off[c] = (uint32_t)((row * K + (((lane % SLOTS) ^ row_swz(row)) * 8)) * 2);
  }
  // the loads of step kt into the stage at st (a step past the last one
  // reloads the last, so that the count of loads in flight stays fixed)
  auto issue = [&](int kt, uint8_t* st) {
    const uint32_t kbyte = (uint32_t)((kt < KT ? kt : KT - 1) * BK * 2);
#pragma unroll
    for (int c = 0; c < A_LOADS; ++c) load_lds16(ra, st + (wave * A_LOADS + c) * 1024, a_off[c], kbyte);
#pragma unroll
    for (int c = 0; c < B_LOADS; ++c)
      load_lds16(rb, st + A_BYTES + (wave * B_LOADS + c) * 1024, b_off[c], kbyte);
  };

  f32x16 acc[MI][NJ_];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ_; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int r32 = lane & 31, hi = lane >> 5, sw = row_swz(r32);
  const int a_row0 = (wm * WR + r32) * ROWB;
  const int b_row0 = A_BYTES + (wn * WCOLS + r32) * ROWB;
  // fragments of NB k-steps: two whole steps where the registers allow it, so
  // that a step's LDS reads run a step ahead of its MFMAs, else two k-steps
  constexpr bool WHOLE = KS * (MI + NJ_) * 8 + MI * NJ_ * 16 + 48 <= (NW <= 4 ? 512 : 256);
  constexpr int NB = WHOLE ? 2 * KS : 2;
  frag fx[NB][MI], fw[NB][NJ_];
  auto read = [&](const uint8_t* st, int kk, int to) {
    const int so = (((kk * 2 + hi) ^ sw) * 16);
#pragma unroll
    for (int j = 0; j < NJ_; ++j) fw[to][j] = *reinterpret_cast<const frag*>(st + b_row0 + j * 32 * ROWB + so);
#pragma unroll
    for (int i = 0; i < MI; ++i) fx[to][i] = *reinterpret_cast<const frag*>(st + a_row0 + i * 32 * ROWB + so);
  };
  auto mfmas = [&](int from) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ_; ++j) acc[i][j] = Mfma<T>::run(fw[from][j], fx[from][i], acc[i][j]);
  };
  // nr LDS reads and nl loads spread over nm MFMAs: issued together, the loads
  // of all waves fill the address queue and hold the MFMAs back
  auto interleave = [](auto nm, auto nr, auto nl) {
#pragma unroll
    for (int g = 0; g < nm(); ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
      for (int n = g * nr() / nm(); n < (g + 1) * nr() / nm(); ++n) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
      for (int n = g * nl() / nm(); n < (g + 1) * nl() / nm(); ++n) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
  };
  auto barrier_landed = [&]() {  // all but the newest NS - 2 steps' loads have landed
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((NS_ - 2) * LPS));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  int cur = 0;  // the stage of step kt
  // step kt, h = kt & 1: the barrier means that every wave has read all of its
  // stage, and that step kt+1 has landed
  auto step = [&](int kt, int h) {
    uint8_t* st = smem_raw + cur * STAGE_BYTES;
    cur = cur + 1 == NS_ ? 0 : cur + 1;
    if constexpr (!WHOLE) {
#pragma unroll
      for (int kk = 0; kk < KS - 1; ++kk) {
        read(st, kk + 1, (kk + 1) & 1);
        mfmas(kk & 1);
        interleave(std::integral_constant<int, MI * NJ_>(), std::integral_constant<int, MI + NJ_>(),
                   std::integral_constant<int, 0>());
      }
    }
    barrier_landed();
    issue(kt + NS_, st);
    const uint8_t* next = smem_raw + cur * STAGE_BYTES;
    if constexpr (WHOLE) {
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) read(next, kk, (h ^ 1) * KS + kk);
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) mfmas(h * KS + kk);
      interleave(std::integral_constant<int, KS * MI * NJ_>(), std::integral_constant<int, KS * (MI + NJ_)>(),
                 std::integral_constant<int, LPS>());
    } else {
      read(next, 0, 0);
      mfmas((KS - 1) & 1);
      interleave(std::integral_constant<int, MI * NJ_>(), std::integral_constant<int, MI + NJ_>(),
                 std::integral_constant<int, LPS>());
    }
  };

#pragma unroll
  for (int s = 0; s < NS_ - 1; ++s) issue(s, smem_raw + s * STAGE_BYTES);
  barrier_landed();  // step 0 has landed
  issue(NS_ - 1, smem_raw + (NS_ - 1) * STAGE_BYTES);
#pragma unroll
  for (int kk = 0; kk < (WHOLE ? KS : 1); ++kk) read(smem_raw, kk, kk);
  int kt = 0;
  for (; kt + 1 < KT; kt += 2) {
    step(kt, 0);
    step(kt + 1, 1);
  }
  if (kt < KT) step(kt, 0);
  // the last iterations' loads still write to LDS, which the epilogue reuses
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));

  store_tile<EPI, CT, RT, MI, NJ_, BM, NW, WR>(p, acc, m0, p.M, n0, wm, wn, lane, wave, smem_raw, bias, cout, resid, gate);
}

template <typename T, int EPI, typename CT, typename RT, int BM, int WMW, int WNW, int NJ_, int NS_>
__global__ __launch_bounds__(WMW * WNW * 64, 1) void k_gemm_ring(GemmParams p, const uint16_t* __restrict__ bias,
                                                            CT* __restrict__ cout, const RT* __restrict__ resid,
                                                            const float* __restrict__ gate) {
  constexpr int STAGES = NS_ * (BM + WNW * 32 * NJ_) * ROWB;
  constexpr int HD = EPI == EPI_QKV_HEADS_128 ? 128 : 64;
  constexpr int EPI_LDS = EPI == EPI_QKV_HEADS || EPI == EPI_QKV_HEADS_128
                              ? qkv_epi_lds_bytes(BM, HD, WMW * WNW, BM / WMW) : 0;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[STAGES > EPI_LDS ? STAGES : EPI_LDS];
  gemm_ring_tile<T, EPI, CT, RT, BM, WMW, WNW, NJ_, NS_>(p, (int)blockIdx.x, smem, bias, cout, resid, gate);
}

// 256 x 192 tiles with the pipeline of gemm_tile (4 x 2 waves of 64 x 96):
// 1000 x 12288 x 3072 75.8 -> 68.1 us, 2048 x 12288 x 3072 155 -> 138 us, 4000 x
// 3072 x 3072 83.7 -> 75.3 us against the two-stage ring of 32x32x16 MFMAs that
// these tiles had (1.3 us a step in place of 1.45).
template <typename T, int EPI, typename CT, typename RT>
__global__ __launch_bounds__(NWAVES * 64, 1) void k_gemm_192(GemmParams p, const uint16_t* __restrict__ bias,
                                                             CT* __restrict__ cout, const RT* __restrict__ resid,
                                                             const float* __restrict__ gate) {
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * 256 * ROWB + 3 * 192 * ROWB];
  gemm_tile<T, EPI, CT, RT, 256, 192, 4>(p, 0, p.M, (int)blockIdx.x, smem, bias, cout, resid, gate);
}

// One launch, two tile heights: 256-row tiles of rows [0, split) and
// 128-row tiles of rows [split, M).  The first `first_small` workgroups take
// half-height tiles, the next tiles_big the full tiles, the rest the other
// half-height tiles, which come last in dispatch order and fill the CUs the
// last round of full tiles leaves idle.  Half-height tiles first put the
// CUs that run them about half a tile ahead of the others, so that their
// epilogues do not all fall in the same interval.
template <typename T, int EPI, typename CT, typename RT>
__global__ __launch_bounds__(NWAVES * 64, 1) void k_gemm(GemmParams p, int64_t split, int tiles_big,
                                                         int first_small,
                                                         const uint16_t* __restrict__ bias,
                                                         CT* __restrict__ cout,
                                                         const RT* __restrict__ resid,
                                                         const float* __restrict__ gate) {
  constexpr int STAGES = 2 * 256 * ROWB + 3 * B_BYTES;   // the operand stages, which the QKV epilogue uses again
  static_assert(qkv_epi_lds_bytes(256, 128) <= STAGES && NWAVES * 64 * v_row(128) * 2 <= STAGES, "epilogue LDS");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[STAGES];
  const int bx = (int)blockIdx.x;
  if (bx < first_small)
    gemm_tile<T, EPI, CT, RT, 128>(p, split, p.M, bx, smem, bias, cout, resid, gate);
  else if (bx < first_small + tiles_big)
    gemm_tile<T, EPI, CT, RT, 256>(p, 0, split, bx - first_small, smem, bias, cout, resid, gate);
  else
    gemm_tile<T, EPI, CT, RT, 128>(p, split, p.M, bx - tiles_big, smem, bias, cout, resid, gate);
}

template <typename T, int EPI, typename CT, typename RT, int BM, int WMW, int WNW, int NJ_, int NS_>
static hipError_t launch_ring(const GemmParams& p, hipStream_t s) {
  const int64_t tiles = ((p.M + BM - 1) / BM) * (p.N / (WNW * 32 * NJ_));
  hipLaunchKernelGGL((k_gemm_ring<T, EPI, CT, RT, BM, WMW, WNW, NJ_, NS_>), dim3((unsigned)tiles),
                     dim3(WMW * WNW * 64), 0, s, p, p.bias, (CT*)p.c, (const RT*)p.resid, p.gate);
  return hipGetLastError();
}

template <typename T, int EPI, typename CT, typename RT>
static hipError_t launch_t(const GemmParams& p, hipStream_t s) {
  const int tiles_n = p.N / BN;
  constexpr int HD = EPI == EPI_QKV_HEADS ? 64 : EPI == EPI_QKV_HEADS_128 ? 128 : 0;
  const GemmPick pick = gemm_pick(p.M, p.N, p.K, HD);
  const int64_t split = pick.split;
  switch (pick.tile) {
    case G256x128: return launch_ring<T, EPI, CT, RT, 256, 4, 2, 2, 3>(p, s);
    case G128x128: return launch_ring<T, EPI, CT, RT, 128, 2, 2, 2, 4>(p, s);
    case G64x128: return launch_ring<T, EPI, CT, RT, 64, 2, 2, 2, 3>(p, s);
    case G64x64:
      if constexpr (HD != 128) return launch_ring<T, EPI, CT, RT, 64, 2, 1, 2, 4>(p, s);
      break;
    case G256x192:
      if constexpr (HD == 0) {
        const int64_t tiles = (p.M + 255) / 256 * (p.N / 192);
        hipLaunchKernelGGL((k_gemm_192<T, EPI, CT, RT>), dim3((unsigned)tiles), dim3(NWAVES * 64), 0, s, p, p.bias,
                           (CT*)p.c, (const RT*)p.resid, p.gate);
        return hipGetLastError();
      }
      break;
    case G128x192:
      if constexpr (HD == 0) return launch_ring<T, EPI, CT, RT, 128, 2, 2, 3, 3>(p, s);
      break;
    case G128x96:
      if constexpr (HD == 0) return launch_ring<T, EPI, CT, RT, 128, 4, 1, 3, 4>(p, s);
      break;
    default: break;
  }
  const int64_t big = ((split + 255) / 256) * tiles_n;
  const int64_t small = ((p.M - split + 127) / 128) * tiles_n;
  // Up to 96 half-height tiles first (a multiple of 8, so that each set of
  // tiles keeps its XCD-aware order) for the gated-residual epilogue at
  // short K (the out-projection), whose epilogue is a large share of a tile.
  // Measured with none, 96 and 192 first, us: 17776 x 3072 x 3072 343, 328, 330;
  // 18432 rows 347, 330, 339; 9216 x 4096 x 4096 297, 285, 286; 13000 x 3072 x
  // 1024 128, 119, 124; 57224 x 4096 x 4096 the same; at K = 12288 1074, 1101, 1091,
  // and with the other epilogues no faster.  The dispatch order changes no
  // result: every tile sums its K products in the same order.
  const int first_small =
      (EPI == XEMA_EPI_GATED_RESIDUAL && p.K <= 4096) ? (int)(std::min<int64_t>(small, 96) & ~7) : 0;
  hipLaunchKernelGGL((k_gemm<T, EPI, CT, RT>), dim3((unsigned)(big + small)), dim3(NWAVES * 64), 0, s, p,
                     split, (int)big, first_small, p.bias, (CT*)p.c, (const RT*)p.resid, p.gate);
  return hipGetLastError();
}

hipError_t launch_gemm(const GemmParams& p, hipStream_t s) {
  if (p.M <= 0) return hipSuccess;
  const bool h = p.dtype == XEMA_F16;
  switch (p.epilogue) {
    case XEMA_EPI_BIAS:
    case XEMA_EPI_BIAS_GELU: {
      const bool gelu = p.epilogue == XEMA_EPI_BIAS_GELU;
      const bool ch = p.c_dtype == XEMA_F16;
      if (h && ch && gelu) return launch_t<f16, XEMA_EPI_BIAS_GELU, f16, float>(p, s);
      if (h && ch) return launch_t<f16, XEMA_EPI_BIAS, f16, float>(p, s);
      if (h && gelu) return launch_t<f16, XEMA_EPI_BIAS_GELU, bf16, float>(p, s);
      if (h) return launch_t<f16, XEMA_EPI_BIAS, bf16, float>(p, s);
      if (ch && gelu) return launch_t<bf16, XEMA_EPI_BIAS_GELU, f16, float>(p, s);
      if (ch) return launch_t<bf16, XEMA_EPI_BIAS, f16, float>(p, s);
      if (gelu) return launch_t<bf16, XEMA_EPI_BIAS_GELU, bf16, float>(p, s);
      return launch_t<bf16, XEMA_EPI_BIAS, bf16, float>(p, s);
    }
    case XEMA_EPI_GATED_RESIDUAL: {
      const bool rf = p.resid_dtype == XEMA_F32;
      if (h && rf) return launch_t<f16, XEMA_EPI_GATED_RESIDUAL, float, float>(p, s);
      if (h) return launch_t<f16, XEMA_EPI_GATED_RESIDUAL, float, uint16_t>(p, s);
      if (rf) return launch_t<bf16, XEMA_EPI_GATED_RESIDUAL, float, float>(p, s);
      return launch_t<bf16, XEMA_EPI_GATED_RESIDUAL, float, uint16_t>(p, s);
    }
    case EPI_QKV_HEADS:
      if (h) return hipErrorInvalidValue;
      return launch_t<bf16, EPI_QKV_HEADS, f16, float>(p, s);
    case EPI_QKV_HEADS_128:
      if (h) return hipErrorInvalidValue;
      return launch_t<bf16, EPI_QKV_HEADS_128, f16, float>(p, s);
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace xema
