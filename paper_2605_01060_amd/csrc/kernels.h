// Host-side launchers of the gfx950 kernels.  Every launcher assumes its
// arguments were checked by the caller (shapes, alignment, index ranges) and
// returns the launch status.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace surge {

// Copies n16 16-byte units of pinned, device-mapped host memory to the
// device in a kernel: one launch for a chunk's whole metadata.
hipError_t launch_upload(const void* pinned, void* dst, int64_t n16, hipStream_t stream);

// x_t = LN(word[id_t] + pos[t - cu_i]) for every token.  tokens [T], items
// the row blocks (device); out bf16 [T, d].  Out-of-vocabulary IDs are
// gathered as ID 0 and set *err = 1.  n_cus: compute units of the device.
hipError_t launch_embed_ln(const int32_t* tokens, const RowBlock* items, int n_items,
                           const uint16_t* word, const uint16_t* pos, const float* gamma,
                           const float* beta, float eps, int vocab, int d, uint16_t* out, int* err,
                           int n_cus, hipStream_t stream);

// Y[M, N] = epi(X[M, K] W^T + b), W stored [N, K] (out, in), bf16 in/out.
// Requires N % 128 == 0, K % 64 == 0, M >= 1.
//   EPI_BIAS          y = acc + b
//   EPI_BIAS_GELU     y = GELU(acc + b)
//   EPI_BIAS_RESIDUAL y = acc + b + R
// LayerNorm folded into its neighbours (post-LN encoder, LN(x) = g (x - mu)
// rstd + beta per row of x):
//   EPI_FOLD          X holds raw rows x (K features) whose per-row
//                     LayerNorm factors are in ex.rows_in; W was built as W diag(g)
//                     and b as b + W beta, and ex.col_s[n] = sum_k W'[n][k],
//                     so y = rstd (acc - mu col_s) + b = LN(x) W^T + b;
//   EPI_FOLD_GELU     the same, then GELU;
//   EPI_RES_STATS     y = acc + b + R, and the per-row statistics of y go
//                     to ex.stats_out;
//   EPI_LNRES_STATS   y = acc + b + LN(R) with R's LayerNorm factors in
//                     ex.rows_in and LN's g, beta in ex.gamma, ex.beta; the
//                     statistics of y go to ex.stats_out.
// Row statistics are partials over linear_stats_width(M, N) = 64
// consecutive features in every tile configuration: float2 (mean, variance)
// at [p * M + row], p < N / 64;
// launch_ln_rows turns them into the per-row LayerNorm factors
// float2 (rstd, -mean * rstd) at [row].
enum LinearEpilogue {
  EPI_BIAS = 0,
  EPI_BIAS_GELU = 1,
  EPI_BIAS_RESIDUAL = 2,
  EPI_FOLD = 3,
  EPI_FOLD_GELU = 4,
  EPI_RES_STATS = 5,
  EPI_LNRES_STATS = 6,
};
struct LinearExtra {
  const float2* rows_in = nullptr;   // LayerNorm factors of X's rows (FOLD) or R's rows (LNRES)
  float2* stats_out = nullptr;       // partials of Y's rows (RES_STATS, LNRES_STATS)
  const float* col_s = nullptr;      // [N] (FOLD)
  const float* gamma = nullptr;      // [N] (LNRES)
  const float* beta = nullptr;       // [N] (LNRES)
  int n_cus = 0;                     // compute units of the device
  // Where linear_merges_stats says so, rows_in may be NULL and the factors
  // are merged from the statistics partials by the tiles that need them.
  const float2* stats_in = nullptr;
  int parts_in = 0;
  float eps = 0.0f;
};
constexpr int RING_MAX_PARTS = 16;  // most partials per row that a tile merges
hipError_t launch_linear(const uint16_t* X, const uint16_t* W, const float* bias, const uint16_t* R,
                         uint16_t* Y, int64_t M, int N, int K, int epi, const LinearExtra& ex,
                         hipStream_t stream);
// Whether an [M, N] linear layer can merge its input's (or residual's) row
// statistics, `parts` partials a row, by itself (ex.stats_in), so that
// launch_ln_rows need not run before it.
bool linear_merges_stats(int64_t M, int N, int K, int parts, int n_cus);
// The tile of an [M, N] layer's launch on a device of n_cus compute units,
// rows << 16 | features (see surge_op_linear_tile).
int linear_tile(int64_t M, int N, int K, int n_cus);
// Sets *n_cus to the current device's compute units unless it is positive.
hipError_t resolve_cus(int* n_cus);
// Features per statistics partial written by launch_linear for an [M, N]
// output (the width of one wave's slice of a tile).
int linear_stats_width(int64_t M, int N);

// Packed varlen multi-head self-attention.  qkv bf16 [T, 3 H dh] (Q | K | V
// column blocks, head h at columns h*dh of each), out bf16 [T, H dh].
// Attention runs within each text only.  dh is 32 or 64.  items: the row
// blocks (device).  n_cus: compute units of the device.
hipError_t launch_attention(const uint16_t* qkv, uint16_t* out, const RowBlock* items, int n_items,
                            int n_heads, int d_head, int n_cus, hipStream_t stream);

// Per-row LayerNorm factors rows[m] = (rstd, -mean * rstd) from `parts`
// equal-width statistics partials stats[p * M + m] = (mean, variance).
hipError_t launch_ln_rows(const float2* stats, int parts, int64_t M, float eps, float2* rows,
                          hipStream_t stream);

// y = LN(x) per row of d (d % 8 == 0, d <= 1024), bf16 in/out.
hipError_t launch_layernorm(const uint16_t* x, const float* gamma, const float* beta, float eps,
                            uint16_t* y, int64_t M, int d, hipStream_t stream);

// e_i = mean of text i's rows of x; row i of the output (at dst[i], a device
// pointer to d floats, or with dst == NULL at out + i d) =
// e_i / max(||e_i||, 1e-12).  With rows != NULL the
// rows of x are raw and LayerNorm(gamma, beta) is applied to each first,
// from its factors rows[t] = (rstd, -mean * rstd).
hipError_t launch_pool_l2_scatter(const uint16_t* x, const int32_t* cu, int n_texts,
                                  const uint64_t* dst, float* out, int d, const float2* rows,
                                  const float* gamma, const float* beta, hipStream_t stream);

}  // namespace surge
