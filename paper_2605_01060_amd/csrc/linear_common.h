// Shared by the linear-layer kernels: the per-output finish of every
// epilogue and the width of a row-statistics partial.
#pragma once

#include "device_common.h"
#include "kernels.h"

namespace surge {

constexpr int STATS_WIDTH = 64;  // features per row-statistics partial

// One row's statistics partial: the sums of the rounded outputs, four
// features at a time, and the (mean, variance) they end in.
__device__ __forceinline__ void row_stats_add(uint2 out, float& s, float& q) {
  const float v0 = __uint_as_float(out.x << 16), v1 = __uint_as_float(out.x & 0xffff0000u);
  const float v2 = __uint_as_float(out.y << 16), v3 = __uint_as_float(out.y & 0xffff0000u);
  s += (v0 + v1) + (v2 + v3);
  q = fmaf(v0, v0, fmaf(v1, v1, fmaf(v2, v2, fmaf(v3, v3, q))));
}
__device__ __forceinline__ float2 row_stats_finish(float s, float q) {
  constexpr float inv_w = 1.0f / (float)STATS_WIDTH;
  const float mean = s * inv_w;
  return make_float2(mean, fmaxf(q * inv_w - mean * mean, 0.0f));
}

// Finishes four consecutive features of one output row and rounds them to
// bf16: bias (or the folded LayerNorm rs * a + (nm * s + b)), GELU, then
// the residual `res` (LayerNorm-applied as (r rs + nm) g + beta in the
// LNRES mode).
template <int EPI>
__device__ __forceinline__ uint2 finish4(const float (&a)[4], float4 bb, float4 cs, float4 gg,
                                         float4 be, float rs, float nm, uint2 res) {
  constexpr bool FOLD = EPI == EPI_FOLD || EPI == EPI_FOLD_GELU;
  constexpr bool GELU = EPI == EPI_BIAS_GELU || EPI == EPI_FOLD_GELU;
  constexpr bool RES = EPI == EPI_BIAS_RESIDUAL || EPI == EPI_RES_STATS || EPI == EPI_LNRES_STATS;
  constexpr bool LNRES = EPI == EPI_LNRES_STATS;
  float o0, o1, o2, o3;
  if constexpr (FOLD) {
    o0 = fmaf(rs, a[0], fmaf(nm, cs.x, bb.x));
    o1 = fmaf(rs, a[1], fmaf(nm, cs.y, bb.y));
    o2 = fmaf(rs, a[2], fmaf(nm, cs.z, bb.z));
    o3 = fmaf(rs, a[3], fmaf(nm, cs.w, bb.w));
  } else {
    o0 = a[0] + bb.x;
    o1 = a[1] + bb.y;
    o2 = a[2] + bb.z;
    o3 = a[3] + bb.w;
  }
  if constexpr (GELU) {
    o0 = gelu_erf(o0);
    o1 = gelu_erf(o1);
    o2 = gelu_erf(o2);
    o3 = gelu_erf(o3);
  }
  if constexpr (RES) {
    float r0 = __uint_as_float(res.x << 16);
    float r1 = __uint_as_float(res.x & 0xffff0000u);
    float r2 = __uint_as_float(res.y << 16);
    float r3 = __uint_as_float(res.y & 0xffff0000u);
    if constexpr (LNRES) {
      r0 = fmaf(fmaf(r0, rs, nm), gg.x, be.x);
      r1 = fmaf(fmaf(r1, rs, nm), gg.y, be.y);
      r2 = fmaf(fmaf(r2, rs, nm), gg.z, be.z);
      r3 = fmaf(fmaf(r3, rs, nm), gg.w, be.w);
    }
    o0 += r0;
    o1 += r1;
    o2 += r2;
    o3 += r3;
  }
  uint2 out;
  out.x = pack_bf16x2(o0, o1);
  out.y = pack_bf16x2(o2, o3);
  return out;
}

// Tile order.  Workgroups are dispatched round-robin over the 8 XCDs
// (block b runs on XCD b % 8), each with its own 4 MB L2, so the order in
// which one XCD walks its tiles decides what its L2 can reuse.
//   ORDER_ROW_GROUPS: each XCD walks a contiguous eighth of the tile grid in
//     groups of 8 token-row blocks, feature tile outer: a weight tile is
//     reused by 8 row blocks and 8 X row blocks stay resident meanwhile.
//   ORDER_FEATURE_HALVES: the XCDs form 2 feature halves x 4 token-row
//     quarters and each walks its rectangle as above, so an XCD touches half
//     of W (FFN1's 4.7 MB W does not fit one L2, half of it does).  Falls
//     back to ORDER_ROW_GROUPS when the rectangles do not divide evenly.
// The blocks beyond the last full eighth keep their own index.
constexpr int ORDER_ROW_GROUPS = 0;
constexpr int ORDER_FEATURE_HALVES = 1;

template <int ORDER>
__device__ __forceinline__ void tile_coords(int b, int n_tiles, int tiles_n, int* tm, int* tn) {
  const int tiles_m = n_tiles / tiles_n;
  const int xcd = b & 7;
  const int local = b >> 3;
  int t, m_base = 0, n_base = 0, m_cnt = tiles_m, n_cnt = tiles_n;
  if (ORDER == ORDER_FEATURE_HALVES && tiles_n % 2 == 0 && tiles_m % 4 == 0) {
    n_cnt = tiles_n / 2;
    m_cnt = tiles_m / 4;
    n_base = (xcd & 1) * n_cnt;
    m_base = (xcd >> 1) * m_cnt;
    t = local;
  } else {
    const int per_xcd = n_tiles >> 3;
    t = b < (per_xcd << 3) ? xcd * per_xcd + local : b;
  }
  const int grp = t / (8 * n_cnt);
  const int in = t - grp * 8 * n_cnt;
  const int rows = min(8, m_cnt - grp * 8);
  *tn = n_base + in / rows;
  *tm = m_base + grp * 8 + in % rows;
}

// Epilogue region layout: 32 rows x 64 bf16, a row as 16 8-byte units;
// unit u of row r sits at u ^ rsw(r).  The 16 rows of two units that half a
// wave's 8-byte access spans land on distinct banks, and an aligned 16-byte
// pair {2k, 2k+1} stays together (halves swapped when rsw(r) is odd).
__device__ __forceinline__ int rsw(int r) { return (r & 15) ^ ((r >> 4) & 1); }

// Accumulators.  The large tiles multiply with 16x16x32 bf16 MFMAs, A =
// 16 features of W and B = 16 tokens of X, so acc[i][j] register r of a lane
// holds Y^T at feature 16 i + 4 (lane / 16) + r, token 16 j + lane % 16: each
// lane owns four consecutive features of one row per accumulator.  (On
// normal data the card runs these loops at its power limit, and 16x16x32
// does 13 % more work per watt than 32x32x16: a register-only loop measured
// 2,077 against 1,830 TFLOP/s, 2,464 against 2,497 on zeros.  The two give
// the same bits.)
typedef f32x4 Acc;
__device__ __forceinline__ Acc mma(bf16x8 w, bf16x8 x, Acc c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x, c, 0, 0, 0);
}

// Row statistics of 64 features x 32 tokens: s[jj], q[jj] are a lane's sums
// over its 16 features of token 16 jj + lane % 16 (row_stats_add in feature
// order).  The four lanes of a token add up as (0 + 1) + (2 + 3); lane
// 16 jj + token (lanes 0 .. 31) ends with that token's totals.
__device__ __forceinline__ float2 row_stats_sum(const float (&s)[2], const float (&q)[2], int lane) {
  const bool odd = lane & 16;
  float a = odd ? s[1] : s[0], b = odd ? q[1] : q[0];
  a += __shfl_xor(odd ? s[0] : s[1], 16, 64);
  b += __shfl_xor(odd ? q[0] : q[1], 16, 64);
  a += __shfl_xor(a, 32, 64);
  b += __shfl_xor(b, 32, 64);
  return row_stats_finish(a, b);
}

// A wave's part of a tile's epilogue, in passes over its own 4 KB LDS region
// (no other wave touches it, so no barrier is needed).  Pass (j, ip) covers
// 32 token rows (accumulators 2j, 2j+1) and 64 features (accumulators 4ip ..
// 4ip+3), which is exactly one row-statistics partial; a lane's accumulator
// is unit 4 (i % 4) + lane/16 of a region row.  Per pass:
//   1. (residual modes) the pass's R rows, loaded for all passes with
//      16-byte coalesced loads before the first, go into the region;
//   2. each lane finishes its accumulators (reading its residual units
//      back), rounds once to bf16 and writes the region; the statistics
//      modes also sum the rounded values of its rows;
//   3. the region is stored as whole 128-byte row segments.
// slot16(r, c): 16-byte slot c of the 8 of region row r.  vec(v, q): the
// tile's per-feature vector v at the wave's features 4q .. 4q+3.  rows(r):
// the LayerNorm factors of the wave's row r.
template <int TJ, int TI, int EPI, class Slot, class Vec, class Rows>
__device__ __forceinline__ void store_tile(const Acc (&acc)[TI][TJ], Slot slot16, Vec vec, Rows rows,
                                           const uint16_t* __restrict__ R,
                                           uint16_t* __restrict__ Y, int mw, int nw, int M, int N,
                                           int lane, const LinearExtra& ex) {
  constexpr bool FOLD = EPI == EPI_FOLD || EPI == EPI_FOLD_GELU;
  constexpr bool RES = EPI == EPI_BIAS_RESIDUAL || EPI == EPI_RES_STATS || EPI == EPI_LNRES_STATS;
  constexpr bool LNRES = EPI == EPI_LNRES_STATS;
  constexpr bool STATS = EPI == EPI_RES_STATS || EPI == EPI_LNRES_STATS;
  constexpr int PI = TI / 4;             // 64-feature groups
  constexpr int NP = (TJ / 2) * PI;      // passes
  static_assert(TI % 4 == 0 && TJ % 2 == 0, "epilogue passes are 32 rows x 64 features");
  const int l16 = lane & 15;
  const int lq = lane >> 4;
  auto cell8 = [&](int r, int u) -> uint2* { return reinterpret_cast<uint2*>(slot16(r, 0)) + u; };
  const int cr = lane >> 3;  // row within the 8 rows of one coalesced access
  const int cp = lane & 7;   // 16-byte pair within a row

  u32x4 rv[RES ? NP : 1][4];
  if constexpr (RES) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int j = p / PI, ip = p % PI;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int m = min(mw + j * 32 + it * 8 + cr, M - 1);
        rv[p][it] = __builtin_nontemporal_load(
            reinterpret_cast<const u32x4*>(R + (size_t)m * N + (nw + ip * 64 + 8 * cp)));
      }
    }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int j = p / PI, ip = p % PI;
    if constexpr (RES) {
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int r = it * 8 + cr;
        const int ph = (2 * cp) ^ rsw(r);  // physical unit of logical unit 2cp
        u32x4 v = rv[p][it];
        if (ph & 1) v = u32x4{v[2], v[3], v[0], v[1]};
        *slot16(r, ph >> 1) = v;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    float2 rf[2];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) rf[jj] = rows(j * 32 + jj * 16 + l16);
    float st_s[2] = {0.0f, 0.0f}, st_q[2] = {0.0f, 0.0f};
#pragma unroll
    for (int ii = 0; ii < 4; ++ii) {
      const int i = 4 * ip + ii;
      const int fq = 4 * i + lq;  // float4 index within the wave's features
      const float4 bb = vec(0, fq);
      float4 cs = {0.0f, 0.0f, 0.0f, 0.0f}, gg = cs, be = cs;
      if constexpr (FOLD) cs = vec(1, fq);
      if constexpr (LNRES) {
        gg = vec(1, fq);
        be = vec(2, fq);
      }
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int r = jj * 16 + l16;
        uint2& cell = *cell8(r, (4 * ii + lq) ^ rsw(r));
        const Acc& v = acc[i][2 * j + jj];
        const float a[4] = {v[0], v[1], v[2], v[3]};
        const uint2 out =
            finish4<EPI>(a, bb, cs, gg, be, rf[jj].x, rf[jj].y, RES ? cell : uint2{0u, 0u});
        cell = out;
        if constexpr (STATS) row_stats_add(out, st_s[jj], st_q[jj]);
      }
    }
    if constexpr (STATS) {
      const float2 st = row_stats_sum(st_s, st_q, lane);
      const int m = mw + j * 32 + (lane & 31);
      if (lane < 32 && m < M) ex.stats_out[(size_t)(nw / STATS_WIDTH + ip) * M + m] = st;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // region written by all lanes
    u32x4 ov[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int r = it * 8 + cr;
      const int ph = (2 * cp) ^ rsw(r);
      ov[it] = *slot16(r, ph >> 1);
      if (ph & 1) ov[it] = u32x4{ov[it][2], ov[it][3], ov[it][0], ov[it][1]};
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // region free for the next pass
    // Everything issued before the tile's first store is done by here: the
    // copies in flight retire before the stores and need not wait for them.
    if (p == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int m = mw + j * 32 + it * 8 + cr;
      if (m < M)
        __builtin_nontemporal_store(
            ov[it], reinterpret_cast<u32x4*>(Y + (size_t)m * N + (nw + ip * 64 + 8 * cp)));
    }
  }
}

// Tiles of the small-token-count kernel (linear_ring.hip).
enum RingTile { RING_NONE, RING_32x64, RING_64x64, RING_64x128 };
hipError_t launch_linear_ring(RingTile tile, const uint16_t* X, const uint16_t* W,
                              const float* bias, const uint16_t* R, uint16_t* Y, int64_t M, int N,
                              int K, int epi, const LinearExtra& ex, hipStream_t stream);

// rows x 256 tiles, rows 256 or 192 (linear_wide.hip), over the first
// N / 256 * 256 features.
hipError_t launch_linear_wide(int rows, const uint16_t* X, const uint16_t* W, const float* bias,
                              const uint16_t* R, uint16_t* Y, int64_t M, int N, int K, int epi,
                              const LinearExtra& ex, hipStream_t stream);

}  // namespace surge
