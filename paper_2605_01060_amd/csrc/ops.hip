// Stage-level entry points: one kernel of the encode path on caller buffers.
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "internal.h"
#include "kernels.h"
#include "surge_ops.h"

using namespace surge;

#define HIP_TRY(expr)                                                                     \
  do {                                                                                    \
    hipError_t e_ = (expr);                                                               \
    if (e_ != hipSuccess)                                                                 \
      return fail(e_ == hipErrorOutOfMemory ? SURGE_ERR_OUT_OF_MEMORY : SURGE_ERR_DEVICE, \
                  "%s failed: %s", #expr, hipGetErrorString(e_));                         \
  } while (0)

namespace {

// Device memory freed on scope exit, with the host data copied into it on
// `stream`.  A call waits for its stream before it returns; one that fails
// before that (`pending`) waits here, so that neither side of the copy is
// freed under it.
struct DeviceBuf {
  std::vector<uint32_t> host;
  void* ptr = nullptr;
  hipStream_t stream = nullptr;
  bool pending = false;
  ~DeviceBuf() {
    if (pending) (void)hipStreamSynchronize(stream);
    if (ptr) hipFree(ptr);
  }
  hipError_t wait() {
    const hipError_t e = hipStreamSynchronize(stream);
    pending = false;
    return e;
  }
};

surge_status check_cu(int64_t n_texts, const int64_t* cu, int64_t max_len) {
  if (n_texts < 1) return fail(SURGE_ERR_INVALID_ARGUMENT, "n_texts=%lld < 1", (long long)n_texts);
  if (!cu) return fail(SURGE_ERR_INVALID_ARGUMENT, "cu_seqlens is NULL");
  if (cu[0] != 0) return fail(SURGE_ERR_INVALID_ARGUMENT, "cu_seqlens[0] != 0");
  for (int64_t i = 0; i < n_texts; ++i) {
    const int64_t L = cu[i + 1] - cu[i];
    if (L < 1 || L > max_len)
      return fail(SURGE_ERR_INVALID_ARGUMENT, "text %lld length %lld outside [1, %lld]",
                  (long long)i, (long long)L, (long long)max_len);
  }
  if (cu[n_texts] > (int64_t)INT32_MAX) return fail(SURGE_ERR_INVALID_ARGUMENT, "too many tokens");
  return SURGE_OK;
}

// One device block of the buffer's host words and one copy on the stream.
surge_status upload(DeviceBuf* buf, hipStream_t s) {
  HIP_TRY(hipMalloc(&buf->ptr, buf->host.size() * 4));
  buf->stream = s;
  buf->pending = true;
  HIP_TRY(hipMemcpyAsync(buf->ptr, buf->host.data(), buf->host.size() * 4, hipMemcpyHostToDevice, s));
  return SURGE_OK;
}

// The row blocks of a checked cu_seqlens, after `head` words of zeros.
surge_status upload_items(int64_t n_texts, const int64_t* cu, int head, DeviceBuf* buf, int* n_items,
                          hipStream_t s) {
  const int64_t n = count_row_blocks(cu, n_texts);
  *n_items = (int)n;
  buf->host.resize((size_t)(head + 2 * n));
  fill_row_blocks(cu, n_texts, (RowBlock*)(buf->host.data() + head));
  return upload(buf, s);
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// Scratch of surge_op_linear_ln_noalloc: the per-row LayerNorm factors of at
// most kScratchRows rows (4 MiB), held by every GPU the library runs on until
// the process ends.  In host code `scratch` names a host-side stand-in, not
// device memory: host code uses only the per-device address obtained from
// hipGetSymbolAddress below.
constexpr int64_t kScratchRows = 1 << 19;
static __device__ __align__(256) float2 scratch[kScratchRows];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float2* g_scratch_ptr[kMaxDevices] = {};

// The device address of the current device's scratch, looked up once per
// device with that device current.
surge_status scratch_address(float2** out) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices)
    return fail(SURGE_ERR_DEVICE, "device index %d outside [0, %d)", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(SURGE_ERR_DEVICE, "hipGetSymbolAddress returned NULL");
    g_scratch_ptr[dev] = (float2*)p;
  }
  *out = g_scratch_ptr[dev];
  return SURGE_OK;
}

}  // namespace

extern "C" {

surge_status surge_op_embed_ln(int64_t n_texts, const int64_t* cu, const int32_t* d_tokens,
                               const uint16_t* d_word, int32_t vocab, const uint16_t* d_pos,
                               int32_t max_pos, const float* d_gamma, const float* d_beta,
                               float eps, int32_t d, uint16_t* d_out, void* hip_stream) {
  clear_error();
  if (d < 128 || d > 1024 || d % 128) return fail(SURGE_ERR_INVALID_ARGUMENT, "d=%d", d);
  if (vocab < 1 || max_pos < 1) return fail(SURGE_ERR_INVALID_ARGUMENT, "vocab/max_pos < 1");
  if (!d_tokens || !d_word || !d_pos || !d_gamma || !d_beta || !d_out)
    return fail(SURGE_ERR_INVALID_ARGUMENT, "NULL device pointer");
  if (!aligned16(d_word) || !aligned16(d_pos) || !aligned16(d_gamma) || !aligned16(d_beta) ||
      !aligned16(d_out))
    return fail(SURGE_ERR_INVALID_ARGUMENT, "device buffers must be 16-byte aligned");
  surge_status st = check_cu(n_texts, cu, std::min(max_pos, 4096));
  if (st != SURGE_OK) return st;
  hipStream_t s = (hipStream_t)hip_stream;
  int n_cus = 0, n_items = 0;
  HIP_TRY(resolve_cus(&n_cus));
  DeviceBuf meta;  // the error flag (and a word of padding), then the row blocks
  st = upload_items(n_texts, cu, 2, &meta, &n_items, s);
  if (st != SURGE_OK) return st;
  HIP_TRY(launch_embed_ln(d_tokens, (const RowBlock*)((int32_t*)meta.ptr + 2), n_items, d_word, d_pos,
                          d_gamma, d_beta, eps, vocab, d, d_out, (int*)meta.ptr, n_cus, s));
  int flag = 0;
  HIP_TRY(hipMemcpyAsync(&flag, meta.ptr, sizeof(int), hipMemcpyDeviceToHost, s));
  HIP_TRY(meta.wait());
  if (flag) return fail(SURGE_ERR_INVALID_ARGUMENT, "a token ID outside [0, vocab) was read as 0");
  return SURGE_OK;
}

surge_status surge_op_linear(int64_t M, int32_t N, int32_t K, const uint16_t* d_x,
                             const uint16_t* d_w, const float* d_bias, const uint16_t* d_res,
                             int32_t epilogue, uint16_t* d_y, void* hip_stream) {
  clear_error();
  if (M < 1 || M > (int64_t)INT32_MAX) return fail(SURGE_ERR_INVALID_ARGUMENT, "M=%lld", (long long)M);
  if (N < 128 || N % 128) return fail(SURGE_ERR_INVALID_ARGUMENT, "N=%d not a multiple of 128", N);
  if (K < 64 || K % 64) return fail(SURGE_ERR_INVALID_ARGUMENT, "K=%d not a multiple of 64", K);
  if (epilogue < 0 || epilogue > 2) return fail(SURGE_ERR_INVALID_ARGUMENT, "epilogue=%d", epilogue);
  if (!d_x || !d_w || !d_bias || !d_y || (epilogue == 2 && !d_res))
    return fail(SURGE_ERR_INVALID_ARGUMENT, "NULL device pointer");
  if (!aligned16(d_x) || !aligned16(d_w) || !aligned16(d_bias) || !aligned16(d_y) ||
      (d_res && !aligned16(d_res)))
    return fail(SURGE_ERR_INVALID_ARGUMENT, "device buffers must be 16-byte aligned");
  hipStream_t s = (hipStream_t)hip_stream;
  LinearExtra ex;
  HIP_TRY(resolve_cus(&ex.n_cus));
  HIP_TRY(launch_linear(d_x, d_w, d_bias, d_res, d_y, M, N, K, epilogue, ex, s));
  HIP_TRY(hipStreamSynchronize(s));
  return SURGE_OK;
}

}  // extern "C"

namespace {

// Argument check shared by surge_op_linear_ln and its no-allocation variant;
// *factors is set when the epilogue reads per-row LayerNorm factors.
surge_status check_linear_ln(int64_t M, int32_t N, int32_t K, const uint16_t* d_x,
                             const uint16_t* d_w, const float* d_bias, const uint16_t* d_res,
                             int32_t epilogue, const float* d_stats_in, int32_t parts_in,
                             const float* d_col_s, const float* d_gamma, const float* d_beta,
                             float eps, float* d_stats_out, uint16_t* d_y, bool* factors) {
  if (M < 1 || M > (int64_t)INT32_MAX) return fail(SURGE_ERR_INVALID_ARGUMENT, "M=%lld", (long long)M);
  if (N < 128 || N % 128) return fail(SURGE_ERR_INVALID_ARGUMENT, "N=%d not a multiple of 128", N);
  if (K < 64 || K % 64) return fail(SURGE_ERR_INVALID_ARGUMENT, "K=%d not a multiple of 64", K);
  if (epilogue < 0 || epilogue > 6) return fail(SURGE_ERR_INVALID_ARGUMENT, "epilogue=%d", epilogue);
  const bool fold = epilogue == EPI_FOLD || epilogue == EPI_FOLD_GELU;
  const bool res = epilogue == EPI_BIAS_RESIDUAL || epilogue >= EPI_RES_STATS;
  const bool lnres = epilogue == EPI_LNRES_STATS;
  const bool stats = epilogue >= EPI_RES_STATS;
  if (!d_x || !d_w || !d_bias || !d_y || (res && !d_res))
    return fail(SURGE_ERR_INVALID_ARGUMENT, "NULL device pointer");
  if ((fold || lnres) && (!d_stats_in || parts_in < 1 || parts_in > 1024))
    return fail(SURGE_ERR_INVALID_ARGUMENT, "stats_in NULL or parts_in=%d outside [1, 1024]",
                parts_in);
  if (fold && !d_col_s) return fail(SURGE_ERR_INVALID_ARGUMENT, "col_s is NULL");
  if (lnres && (!d_gamma || !d_beta)) return fail(SURGE_ERR_INVALID_ARGUMENT, "gamma/beta NULL");
  if (stats && !d_stats_out) return fail(SURGE_ERR_INVALID_ARGUMENT, "stats_out is NULL");
  if ((fold || lnres) && !(eps > 0.0f)) return fail(SURGE_ERR_INVALID_ARGUMENT, "eps must be > 0");
  if (!aligned16(d_x) || !aligned16(d_w) || !aligned16(d_bias) || !aligned16(d_y) ||
      (d_res && !aligned16(d_res)) || (d_col_s && !aligned16(d_col_s)) ||
      (d_gamma && !aligned16(d_gamma)) || (d_beta && !aligned16(d_beta)) ||
      (d_stats_in && ((uintptr_t)d_stats_in & 7u)) || (d_stats_out && ((uintptr_t)d_stats_out & 7u)))
    return fail(SURGE_ERR_INVALID_ARGUMENT, "device buffers must be aligned (16 B; stats 8 B)");
  *factors = fold || lnres;
  return SURGE_OK;
}

// Whether the linear layer merges its input's statistics partials itself, so
// that no row factors are needed.  Not where one of its outputs overlaps the
// partials (statistics updated in place): a tile would write what another
// still has to read, and the row-factor kernel reads them all first.
bool merges_stats(int64_t M, int32_t N, int32_t K, const float* d_stats_in, int32_t parts_in,
                  const float* d_stats_out, const uint16_t* d_y, int n_cus) {
  const uintptr_t in = (uintptr_t)d_stats_in;
  const uint64_t bytes = (uint64_t)M * (uint64_t)parts_in * 8u;
  auto overlaps = [&](const void* p, uint64_t n) {
    return p && (uintptr_t)p < in + bytes && in < (uintptr_t)p + n;
  };
  if (overlaps(d_stats_out, (uint64_t)M * (uint64_t)(N / linear_stats_width(M, N)) * 8u) ||
      overlaps(d_y, (uint64_t)M * (uint64_t)N * 2u))
    return false;
  return linear_merges_stats(M, N, K, parts_in, n_cus);
}

// Enqueue the row factors (when `rows` is not NULL) and the linear layer,
// which merges the partials itself otherwise (merges_stats).
surge_status enqueue_linear_ln(int64_t M, int32_t N, int32_t K, const uint16_t* d_x,
                               const uint16_t* d_w, const float* d_bias, const uint16_t* d_res,
                               int32_t epilogue, const float* d_stats_in, int32_t parts_in,
                               const float* d_col_s, const float* d_gamma, const float* d_beta,
                               float eps, float* d_stats_out, uint16_t* d_y, float2* rows,
                               int n_cus, hipStream_t s) {
  LinearExtra ex;
  ex.n_cus = n_cus;
  ex.stats_out = (float2*)d_stats_out;
  ex.col_s = d_col_s;
  ex.gamma = d_gamma;
  ex.beta = d_beta;
  ex.stats_in = (const float2*)d_stats_in;
  ex.parts_in = parts_in;
  ex.eps = eps;
  if (rows) {
    HIP_TRY(launch_ln_rows((const float2*)d_stats_in, parts_in, M, eps, rows, s));
    ex.rows_in = rows;
  }
  HIP_TRY(launch_linear(d_x, d_w, d_bias, d_res, d_y, M, N, K, epilogue, ex, s));
  return SURGE_OK;
}

}  // namespace

extern "C" {

surge_status surge_op_linear_ln(int64_t M, int32_t N, int32_t K, const uint16_t* d_x,
                                const uint16_t* d_w, const float* d_bias, const uint16_t* d_res,
                                int32_t epilogue, const float* d_stats_in, int32_t parts_in,
                                const float* d_col_s, const float* d_gamma, const float* d_beta,
                                float eps, float* d_stats_out, uint16_t* d_y, void* hip_stream) {
  clear_error();
  bool factors = false;
  surge_status st = check_linear_ln(M, N, K, d_x, d_w, d_bias, d_res, epilogue, d_stats_in,
                                    parts_in, d_col_s, d_gamma, d_beta, eps, d_stats_out, d_y,
                                    &factors);
  if (st != SURGE_OK) return st;
  hipStream_t s = (hipStream_t)hip_stream;
  int n_cus = 0;
  HIP_TRY(resolve_cus(&n_cus));
  DeviceBuf rows;  // per-row LayerNorm factors, freed on return
  if (factors && !merges_stats(M, N, K, d_stats_in, parts_in, d_stats_out, d_y, n_cus))
    HIP_TRY(hipMalloc(&rows.ptr, (size_t)M * 8));
  st = enqueue_linear_ln(M, N, K, d_x, d_w, d_bias, d_res, epilogue, d_stats_in, parts_in, d_col_s,
                         d_gamma, d_beta, eps, d_stats_out, d_y, (float2*)rows.ptr, n_cus, s);
  if (st != SURGE_OK) return st;
  HIP_TRY(hipStreamSynchronize(s));
  return SURGE_OK;
}

surge_status surge_op_linear_ln_noalloc(int64_t M, int32_t N, int32_t K, const uint16_t* d_x,
                                        const uint16_t* d_w, const float* d_bias,
                                        const uint16_t* d_res, int32_t epilogue,
                                        const float* d_stats_in, int32_t parts_in,
                                        const float* d_col_s, const float* d_gamma,
                                        const float* d_beta, float eps, float* d_stats_out,
                                        uint16_t* d_y, void* hip_stream) {
  clear_error();
  bool factors = false;
  surge_status st = check_linear_ln(M, N, K, d_x, d_w, d_bias, d_res, epilogue, d_stats_in,
                                    parts_in, d_col_s, d_gamma, d_beta, eps, d_stats_out, d_y,
                                    &factors);
  if (st != SURGE_OK) return st;
  float2* rows = nullptr;
  if (factors && M > kScratchRows)
    return fail(SURGE_ERR_CAPACITY, "M=%lld rows exceed the %lld rows of the static scratch",
                (long long)M, (long long)kScratchRows);
  int n_cus = 0;
  HIP_TRY(resolve_cus(&n_cus));
  if (factors && !merges_stats(M, N, K, d_stats_in, parts_in, d_stats_out, d_y, n_cus)) {
    st = scratch_address(&rows);
    if (st != SURGE_OK) return st;
  }
  return enqueue_linear_ln(M, N, K, d_x, d_w, d_bias, d_res, epilogue, d_stats_in, parts_in,
                           d_col_s, d_gamma, d_beta, eps, d_stats_out, d_y, rows, n_cus,
                           (hipStream_t)hip_stream);
}

int32_t surge_op_linear_stats_width(int64_t M, int32_t N) { return linear_stats_width(M, N); }

int32_t surge_op_linear_tile(int64_t M, int32_t N, int32_t K, int32_t n_cus) {
  if (M < 1 || M > (int64_t)INT32_MAX || N < 128 || N % 128 || K < 64 || K % 64 || n_cus < 1)
    return 0;
  return linear_tile(M, N, K, n_cus);
}

surge_status surge_op_attention(int64_t n_texts, const int64_t* cu, int32_t n_heads, int32_t d_head,
                                const uint16_t* d_qkv, uint16_t* d_out, void* hip_stream) {
  clear_error();
  if (d_head != 32 && d_head != 64) return fail(SURGE_ERR_INVALID_ARGUMENT, "d_head=%d", d_head);
  if (n_heads < 1 || (n_heads * d_head) % 128)
    return fail(SURGE_ERR_INVALID_ARGUMENT, "n_heads*d_head must be a multiple of 128");
  if (!d_qkv || !d_out) return fail(SURGE_ERR_INVALID_ARGUMENT, "NULL device pointer");
  if (!aligned16(d_qkv) || !aligned16(d_out))
    return fail(SURGE_ERR_INVALID_ARGUMENT, "device buffers must be 16-byte aligned");
  surge_status st = check_cu(n_texts, cu, 4096);
  if (st != SURGE_OK) return st;
  hipStream_t s = (hipStream_t)hip_stream;
  int n_cus = 0, n_items = 0;
  HIP_TRY(resolve_cus(&n_cus));
  DeviceBuf items;
  st = upload_items(n_texts, cu, 0, &items, &n_items, s);
  if (st != SURGE_OK) return st;
  HIP_TRY(launch_attention(d_qkv, d_out, (const RowBlock*)items.ptr, n_items, n_heads, d_head, n_cus,
                           s));
  HIP_TRY(items.wait());
  return SURGE_OK;
}

surge_status surge_op_layernorm(int64_t M, int32_t d, const uint16_t* d_x, const float* d_gamma,
                                const float* d_beta, float eps, uint16_t* d_y, void* hip_stream) {
  clear_error();
  if (M < 1) return fail(SURGE_ERR_INVALID_ARGUMENT, "M < 1");
  if (d < 8 || d > 1024 || d % 8) return fail(SURGE_ERR_INVALID_ARGUMENT, "d=%d", d);
  if (!d_x || !d_gamma || !d_beta || !d_y) return fail(SURGE_ERR_INVALID_ARGUMENT, "NULL pointer");
  if (!aligned16(d_x) || !aligned16(d_gamma) || !aligned16(d_beta) || !aligned16(d_y))
    return fail(SURGE_ERR_INVALID_ARGUMENT, "device buffers must be 16-byte aligned");
  hipStream_t s = (hipStream_t)hip_stream;
  HIP_TRY(launch_layernorm(d_x, d_gamma, d_beta, eps, d_y, M, d, s));
  HIP_TRY(hipStreamSynchronize(s));
  return SURGE_OK;
}

surge_status surge_op_pool_l2(int64_t n_texts, const int64_t* cu, int32_t d, const uint16_t* d_x,
                              float* d_out, void* hip_stream) {
  clear_error();
  if (d < 128 || d > 1024 || d % 128) return fail(SURGE_ERR_INVALID_ARGUMENT, "d=%d", d);
  if (!d_x || !d_out) return fail(SURGE_ERR_INVALID_ARGUMENT, "NULL device pointer");
  if (!aligned16(d_x) || !aligned16(d_out))
    return fail(SURGE_ERR_INVALID_ARGUMENT, "device buffers must be 16-byte aligned");
  surge_status st = check_cu(n_texts, cu, 1 << 16);
  if (st != SURGE_OK) return st;
  hipStream_t s = (hipStream_t)hip_stream;
  DeviceBuf dcu;
  dcu.host.resize((size_t)n_texts + 1);
  for (int64_t i = 0; i <= n_texts; ++i) dcu.host[(size_t)i] = (uint32_t)cu[i];
  st = upload(&dcu, s);
  if (st != SURGE_OK) return st;
  HIP_TRY(launch_pool_l2_scatter(d_x, (const int32_t*)dcu.ptr, (int)n_texts, nullptr, d_out, d,
                                 nullptr, nullptr, nullptr, s));
  HIP_TRY(dcu.wait());
  return SURGE_OK;
}

}  // extern "C"
