// Row-wise, HBM-bound kernels: embedding gather + LayerNorm, LayerNorm, and
// masked mean pooling + L2 normalisation + partition scatter.
//
// A row of d bf16 values is read as d/8 16-byte chunks spread over 16 or 32
// lanes of a wave (at most four chunks per lane for d <= 1024); mean and
// variance are reductions over them in fp32 (two passes over the registers,
// so the variance is taken about the mean).
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace surge {
namespace {

// Sum over the LPR (16 or 32) lanes of a row: four rotations inside 16 lanes
// on the VALU, then the other half.  Every lane ends with the same bits.
template <int LPR>
__device__ __forceinline__ float group_sum(float v) {
  auto rotated = [](float x, auto ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, false));
  };
  v += rotated(v, std::integral_constant<int, 0x128>());  // row_ror:8
  v += rotated(v, std::integral_constant<int, 0x124>());
  v += rotated(v, std::integral_constant<int, 0x122>());
  v += rotated(v, std::integral_constant<int, 0x121>());
  if constexpr (LPR == 32) v += __shfl_xor(v, 16, 64);
  return v;
}

// A lane's chunks gl, gl + LPR, ... of a row's per-feature vector.
template <int LPR, int C>
__device__ __forceinline__ void load_vector(const float* __restrict__ src, int gl, int nch,
                                            float (&v)[C][8]) {
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int ch = min(gl + LPR * c, nch - 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float4 a = reinterpret_cast<const float4*>(src)[2 * ch + h];
      v[c][4 * h] = a.x, v[c][4 * h + 1] = a.y, v[c][4 * h + 2] = a.z, v[c][4 * h + 3] = a.w;
    }
  }
}

// LayerNorm of a row held by LPR lanes (v: in, then overwritten), stored to
// y, nontemporally with STREAM_OUT, where `valid`.
template <int LPR, int C, bool STREAM_OUT>
__device__ __forceinline__ void ln_store(float (&v)[C][8], const float (&ga)[C][8],
                                         const float (&be)[C][8], int gl, int nch, float inv_d,
                                         float eps, bool valid, uint16_t* __restrict__ yrow) {
  float s = 0.0f, sq = 0.0f;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const bool in = gl + LPR * c < nch;
#pragma unroll
    for (int e = 0; e < 8; ++e) s += in ? v[c][e] : 0.0f;
  }
  const float mean = group_sum<LPR>(s) * inv_d;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const bool in = gl + LPR * c < nch;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[c][e] -= mean;
      sq = in ? fmaf(v[c][e], v[c][e], sq) : sq;
    }
  }
  const float rstd = 1.0f / sqrtf(fmaf(group_sum<LPR>(sq), inv_d, eps));
  u32x4* y = reinterpret_cast<u32x4*>(yrow);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = fmaf(v[c][e] * rstd, ga[c][e], be[c][e]);
    const u32x4 packed = __builtin_bit_cast(u32x4, pack8(o));
    if (valid && gl + LPR * c < nch) {
      if constexpr (STREAM_OUT)
        __builtin_nontemporal_store(packed, y + gl + LPR * c);
      else
        y[gl + LPR * c] = packed;
    }
  }
}

// One workgroup per `rows` rows of a work item (a 32-row block of a text),
// so a long text is spread over several workgroups.  LPR lanes take a row,
// C 16-byte chunks each, so a wave works on R = 64 / LPR rows at once and
// keeps its chunks of gamma and beta (8 bytes per feature, twice what the
// tables hold) in registers instead of loading them for every row; a row's
// two reductions are VALU rotations.  A wave loads all its token IDs at once
// (one per lane) and fetches the tables' chunks of its next R rows before it
// normalises the current ones.
//
// Bound by HBM (a byte out per byte gathered); before, one wave took a row:
// a third of its lanes idle at d = 768, gamma and beta loaded per row, and
// twelve LDS shuffles in two chains.  2000 texts of ~54 tokens, us per call
// (20 to 50 of them the host's), one row per wave / this / with STREAM_OUT:
// d = 768 139.7 / 109.7 / 86.9, 384 97 / 69 / 68, 1024 131 / 117 / 112, 128
// 92 / 50 / 48.
template <int LPR, int C, bool STREAM_OUT>
__global__ __launch_bounds__(256) void embed_ln_kernel(
    const int32_t* __restrict__ tokens, const RowBlock* __restrict__ items, int rows,
    const uint16_t* __restrict__ word, const uint16_t* __restrict__ pos,
    const float* __restrict__ gamma, const float* __restrict__ beta, float eps, int vocab, int d,
    uint16_t* __restrict__ out, int* __restrict__ err) {
  constexpr int R = 64 / LPR;
  const RowBlock item = items[blockIdx.x];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int g = lane / LPR;  // this lane's row of the R
  const int gl = lane % LPR;
  const int beg = (int)item.beg;
  const int first = (int)(item.len_block & 127u) * 32 + (int)blockIdx.y * rows + wave * R;
  const int end = min((int)(item.len_block & 127u) * 32 + ((int)blockIdx.y + 1) * rows,
                      (int)(item.len_block >> 7));
  if (first >= end) return;
  // The wave's rows: first + 4 R i + r, r < R, its trip i.
  const int trips = (end - first + 4 * R - 1) / (4 * R);
  const int nch = d >> 3;
  int ids = 0;
  {
    const int p = first + lane / R * (4 * R) + lane % R;  // trip lane / R, row lane % R
    if (lane < trips * R && p < end) {
      ids = tokens[beg + p];
      if (ids < 0 || ids >= vocab) {
        atomicOr(err, 1);
        ids = 0;
      }
    }
  }
  float ga[C][8], be[C][8];
  load_vector<LPR>(gamma, gl, nch, ga);
  load_vector<LPR>(beta, gl, nch, be);
  uint4 w[2][C], q[2][C];
  // Table chunks of the wave's trip i (word rows of its checked IDs, position
  // rows; a group without a row reads the last one's position and ID 0).
  auto fetch = [&](int i, int slot) {
    const int id = __shfl(ids, i * R + g, 64);
    const int p = min(first + 4 * R * i + g, end - 1);
    const uint4* wr = reinterpret_cast<const uint4*>(word + (size_t)id * d);
    const uint4* pr = reinterpret_cast<const uint4*>(pos + (size_t)p * d);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int ch = min(gl + LPR * c, nch - 1);
      w[slot][c] = wr[ch];
      q[slot][c] = pr[ch];
    }
  };
  const float inv_d = 1.0f / (float)d;
  auto row = [&](int i, int slot) {
    float v[C][8];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      float a[8], b[8];
      unpack8(w[slot][c], a);
      unpack8(q[slot][c], b);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[c][e] = a[e] + b[e];
    }
    if (i + 2 < trips) fetch(i + 2, slot);
    const int p = first + 4 * R * i + g;
    ln_store<LPR, C, STREAM_OUT>(v, ga, be, gl, nch, inv_d, eps, p < end,
                                 out + (size_t)(beg + p) * d);
  };
  fetch(0, 0);
  if (trips > 1) fetch(1, 1);
  for (int i = 0; i < trips; i += 2) {
    row(i, 0);
    if (i + 1 < trips) row(i + 1, 1);
  }
}

// 16 bytes per thread from mapped host memory.
__global__ __launch_bounds__(256) void upload_kernel(const uint4* __restrict__ src,
                                                     uint4* __restrict__ dst, int64_t n16) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n16) dst[i] = src[i];
}

// Rows as in the embedding: LPR lanes a row, a wave's trips of R rows each,
// the next trip's chunks fetched before the current rows are normalised (a
// wave reads and writes rows of its own only, so y may be x).  Bound by HBM.
// Against one row per wave, us per call of 100,000 / 300,000 rows (about 12 of
// them the host's): d = 768 78.9 -> 56.1 / 202 -> 161, 384 40.6 -> 34.8 / 124
// -> 77.6, 1024 84.7 -> 70.6 / 222 -> 209, 128 38.7 -> 20.3 / 87.1 -> 33.6.
template <int LPR, int C, bool STREAM_OUT>
__global__ __launch_bounds__(256) void layernorm_kernel(const uint16_t* __restrict__ x,
                                                        const float* __restrict__ gamma,
                                                        const float* __restrict__ beta, float eps,
                                                        uint16_t* __restrict__ y, int64_t M, int d,
                                                        int trips) {
  constexpr int R = 64 / LPR;
  const int lane = threadIdx.x & 63;
  const int gl = lane % LPR;
  const int nch = d >> 3;
  const float inv_d = 1.0f / (float)d;
  int64_t row = ((int64_t)blockIdx.x * trips * 4 + (threadIdx.x >> 6)) * R + lane / LPR;
  uint4 next[C];
  auto fetch = [&](int64_t r) {
    const uint4* xr = reinterpret_cast<const uint4*>(x + (size_t)min(r, M - 1) * d);
#pragma unroll
    for (int c = 0; c < C; ++c) next[c] = xr[min(gl + LPR * c, nch - 1)];
  };
  fetch(row);
  float ga[C][8], be[C][8];
  load_vector<LPR>(gamma, gl, nch, ga);
  load_vector<LPR>(beta, gl, nch, be);
  for (int i = 0; i < trips; ++i, row += 4 * R) {
    float v[C][8];
#pragma unroll
    for (int c = 0; c < C; ++c) unpack8(next[c], v[c]);
    if (i + 1 < trips) fetch(row + 4 * R);
    ln_store<LPR, C, STREAM_OUT>(v, ga, be, gl, nch, inv_d, eps, row < M, y + (size_t)row * d);
  }
}

// One block per text: 2 groups of 128 threads split the text's rows, each
// thread owns one 16-byte column chunk; the norm is a block reduction.
// With LN, x holds raw rows and row t's LayerNorm is applied on the fly:
// rows[t] = (rstd, -mean rstd), and the pooled vector is
// gamma * mean_t(x_t rstd_t - mean_t rstd_t) + beta.
template <bool LN>
__global__ __launch_bounds__(256) void pool_l2_scatter_kernel(const uint16_t* __restrict__ x,
                                                              const int32_t* __restrict__ cu,
                                                              const uint64_t* __restrict__ dst,
                                                              float* __restrict__ out, int d,
                                                              const float2* __restrict__ rows,
                                                              const float* __restrict__ gamma,
                                                              const float* __restrict__ beta) {
  __shared__ float part[128 * 8];
  __shared__ float red[4];
  const int t = blockIdx.x;
  const int c = threadIdx.x & 127;
  const int grp = threadIdx.x >> 7;
  const int beg = cu[t];
  const int L = cu[t + 1] - beg;
  const int nch = d >> 3;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (c < nch) {
    // Unrolled so that several rows' loads are in flight at once (the sum
    // keeps its row order).
#pragma unroll 4
    for (int p = grp; p < L; p += 2) {
      float f[8];
      unpack8(reinterpret_cast<const uint4*>(x + (size_t)(beg + p) * d)[c], f);
      if constexpr (LN) {
        const float2 rf = rows[beg + p];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += fmaf(f[e], rf.x, rf.y);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += f[e];
      }
    }
  }
  if (grp == 1 && c < nch) {
#pragma unroll
    for (int e = 0; e < 8; ++e) part[c * 8 + e] = acc[e];
  }
  __syncthreads();
  float sq = 0.0f;
  if (grp == 0 && c < nch) {
    const float invL = 1.0f / (float)L;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      acc[e] = (acc[e] + part[c * 8 + e]) * invL;
      if constexpr (LN) acc[e] = fmaf(acc[e], gamma[8 * c + e], beta[8 * c + e]);
      sq += acc[e] * acc[e];
    }
  }
  sq = wave_sum(sq);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sq;
  __syncthreads();
  const float norm = sqrtf(red[0] + red[1]);
  const float inv = 1.0f / fmaxf(norm, 1e-12f);
  if (grp == 0 && c < nch) {
    float* row = dst ? reinterpret_cast<float*>(dst[t]) : out + (size_t)t * d;
    float4 a = make_float4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
    float4 b = make_float4(acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv);
    reinterpret_cast<float4*>(row)[2 * c] = a;
    reinterpret_cast<float4*>(row)[2 * c + 1] = b;
  }
}

// Per-row LayerNorm factors from equal-width statistics partials (mean,
// biased variance) at stats[p * M + row]: rows[row] = (rstd, -mean * rstd),
// so that LN(v) = gamma (v rstd - mean rstd) + beta.  MAXP = 16 is the
// encoder's case (d_model / 64 <= 16 partials), MAXP = 0 takes any count.
template <int MAXP>
__global__ __launch_bounds__(256) void ln_rows_kernel(const float2* __restrict__ stats, int parts,
                                                      int64_t M, float eps,
                                                      float2* __restrict__ rows) {
  const int64_t m = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (m >= M) return;
  rows[m] = ln_row_factors<MAXP>([&](int p) { return stats[(size_t)p * M + m]; }, parts, eps);
}

}  // namespace

// 16 lanes a row up to d = 512 (4 rows per wave), then 32 (2 rows): at most
// four chunks per lane.
static int lanes_per_row(int d) { return d <= 512 ? 16 : 32; }
#define SURGE_ROW_LAYOUTS(d, LAUNCH)                                         \
  switch (((d) / 8 + lanes_per_row(d) - 1) / lanes_per_row(d)) {             \
    case 1: LAUNCH(16, 1); break;                                            \
    case 2: LAUNCH(16, 2); break;                                            \
    case 3:                                                                  \
      if (d <= 512) { LAUNCH(16, 3); } else { LAUNCH(32, 3); }               \
      break;                                                                 \
    case 4:                                                                  \
      if (d <= 512) { LAUNCH(16, 4); } else { LAUNCH(32, 4); }               \
      break;                                                                 \
    default: return hipErrorInvalidValue;                                    \
  }

// An output that does not fit the L2s (8 x 4 MB) is stored nontemporally,
// which leaves them to the rows being read; a smaller one stays for the layer
// that reads it next (57 MiniLM texts, 1.5 MB: 271 us per call, 274 with
// nontemporal stores).
constexpr int64_t STREAM_OUT_BYTES = (int64_t)32 << 20;

hipError_t launch_embed_ln(const int32_t* tokens, const RowBlock* items, int n_items,
                           const uint16_t* word, const uint16_t* pos, const float* gamma,
                           const float* beta, float eps, int vocab, int d, uint16_t* out, int* err,
                           int n_cus, hipStream_t stream) {
  if (n_items <= 0) return hipSuccess;
  const int lpr = lanes_per_row(d);
  // Whole 32-row items once they fill the chip (8 workgroups per CU); fewer
  // rows per workgroup, down to one trip of its waves, while they do not.
  int split = 1;
  while (split < lpr / 8 && (int64_t)n_items * split * 2 <= (int64_t)n_cus * 8) split *= 2;
  const bool stream_out = (int64_t)n_items * 32 * d * 2 > STREAM_OUT_BYTES;
#define SURGE_EMBED(L, C)                                                                      \
  if (stream_out)                                                                              \
    hipLaunchKernelGGL((embed_ln_kernel<L, C, true>), dim3(n_items, split), dim3(256), 0, stream, \
                       tokens, items, 32 / split, word, pos, gamma, beta, eps, vocab, d, out, err); \
  else                                                                                         \
    hipLaunchKernelGGL((embed_ln_kernel<L, C, false>), dim3(n_items, split), dim3(256), 0, stream, \
                       tokens, items, 32 / split, word, pos, gamma, beta, eps, vocab, d, out, err)
  SURGE_ROW_LAYOUTS(d, SURGE_EMBED)
#undef SURGE_EMBED
  return hipGetLastError();
}

hipError_t launch_upload(const void* pinned, void* dst, int64_t n16, hipStream_t stream) {
  if (n16 <= 0) return hipSuccess;
  hipLaunchKernelGGL(upload_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, stream,
                     (const uint4*)pinned, (uint4*)dst, n16);
  return hipGetLastError();
}

hipError_t launch_ln_rows(const float2* stats, int parts, int64_t M, float eps, float2* rows,
                          hipStream_t stream) {
  if (M <= 0) return hipSuccess;
  if (parts < 1) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((M + 255) / 256));
  if (parts <= 16)
    hipLaunchKernelGGL(ln_rows_kernel<16>, grid, dim3(256), 0, stream, stats, parts, M, eps, rows);
  else
    hipLaunchKernelGGL(ln_rows_kernel<0>, grid, dim3(256), 0, stream, stats, parts, M, eps, rows);
  return hipGetLastError();
}

hipError_t launch_layernorm(const uint16_t* x, const float* gamma, const float* beta, float eps,
                            uint16_t* y, int64_t M, int d, hipStream_t stream) {
  if (M <= 0) return hipSuccess;
  const int lpr = lanes_per_row(d), rows = 4 * 64 / lpr;  // rows of a workgroup's trip
  // Two trips, for gamma and beta's sake, once they leave 2,048 workgroups:
  // more keep rows of too many places in flight (300,000 rows, 1 / 2 / 3 / 4 /
  // 8 trips, us: d = 1024 220 / 209 / 220 / 236 / 245, 768 164 / 161 / 168 /
  // 174 / 184, 384 75.0 / 77.6 / 78.6 / 79.4 / 81.3).
  const int trips = M >= (int64_t)rows * 4096 ? 2 : 1;
  const dim3 grid((unsigned)((M + rows * trips - 1) / (rows * trips)));
  const bool stream_out = M * d * 2 > STREAM_OUT_BYTES;
#define SURGE_LAYERNORM(L, C)                                                                   \
  if (stream_out)                                                                               \
    hipLaunchKernelGGL((layernorm_kernel<L, C, true>), grid, dim3(256), 0, stream, x, gamma, beta, \
                       eps, y, M, d, trips);                                                    \
  else                                                                                          \
    hipLaunchKernelGGL((layernorm_kernel<L, C, false>), grid, dim3(256), 0, stream, x, gamma,   \
                       beta, eps, y, M, d, trips)
  SURGE_ROW_LAYOUTS(d, SURGE_LAYERNORM)
#undef SURGE_LAYERNORM
  return hipGetLastError();
}

hipError_t launch_pool_l2_scatter(const uint16_t* x, const int32_t* cu, int n_texts,
                                  const uint64_t* dst, float* out, int d, const float2* rows,
                                  const float* gamma, const float* beta, hipStream_t stream) {
  if (n_texts <= 0) return hipSuccess;
  if (rows)
    hipLaunchKernelGGL(pool_l2_scatter_kernel<true>, dim3(n_texts), dim3(256), 0, stream, x, cu,
                       dst, out, d, rows, gamma, beta);
  else
    hipLaunchKernelGGL(pool_l2_scatter_kernel<false>, dim3(n_texts), dim3(256), 0, stream, x, cu,
                       dst, out, d, rows, gamma, beta);
  return hipGetLastError();
}

}  // namespace surge
