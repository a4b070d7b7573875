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

// Tiles of the small-token-count kernel (linear_ring.hip).
enum RingTile { RING_NONE, RING_32x64, RING_64x64, RING_64x128 };
hipError_t launch_linear_ring(RingTile tile, const uint16_t* X, const uint16_t* W,
                              const float* bias, const uint16_t* R, uint16_t* Y, int64_t M, int N,
                              int K, int epi, const LinearExtra& ex, hipStream_t stream);

}  // namespace surge
