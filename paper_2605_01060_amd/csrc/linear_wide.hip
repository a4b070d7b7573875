// Token-major linear layers of large chunks (gfx950): Y = epi(X W^T + b) in
// 256 x 256 tiles (192 x 256 where those leave fewer CUs idle), one persistent
// 8-wave workgroup per CU, each wave a 64 token x 128 feature (96 x 64)
// sub-tile of 16x16x32 bf16 MFMAs.
//
// What bounds it: the power limit and late operand copies.  On normal data
// (K = 3072, TFLOP/s) a loop that gave each copy one K stage to arrive ran at
// 1,160, with copies that all hit the L2 at 1,335 and without copies at
// 1,600; on zeros, where power does not count, 1,390, 1,918 and 1,966.  Hence
// the MFMA that needs less power (linear_common.h) and a schedule that gives
// copies more time.  128 KB of LDS hold two 64-wide stages of a tile whatever
// the schedule, so this one frees LDS earlier: a wave keeps a whole stage's W
// fragments in registers;
// a stage runs as two phases, the wave's first and then its other token rows
// against the same W fragments, and each W fragment is replaced by the
// next stage's right after its last MFMA.  So
//   - W and the phase-0 rows of stage s are read out by the end of stage s-1,
//     and their LDS takes stage s+2 from there on (barrier B, placed after
//     the first four MFMAs of stage s so that no wave waits for its reads);
//   - the phase-1 rows of stage s are read out by the middle of stage s
//     (barrier A, between the phases), and theirs takes stage s+2.
// Every copy has one and a half stages to arrive, and the MFMAs after either
// barrier find their operands in registers.  The copies are spread over the
// MFMAs, since a burst of them blocks the issue of everything behind it.
//
// The copy stream runs on across tile boundaries.  Only the phase-1 rows of
// the next tile's second stage are held back: their LDS and 16 KB (24 KB)
// beside the stages are the waves' epilogue regions.  The accumulators see the
// same K order as every other tile shape.
//
// Measured against the loop of one-stage tolerance on 32x32x16 MFMAs that it
// replaces (M = 262,144, us, normal data): QKV 907 -> 849, FFN2 1,151 ->
// 1,066, FFN1 1,436 -> 1,298, O-projection 391 -> 373.
//
// Two things that the schedule needs, and what they measure:
//   - No instance may spill: a spilled address that a copy uses brings a wait
//     for every copy in flight into the K loop.  One register did so in FFN1,
//     FFN2 and the O-projection; without it, on zeros, where power does not
//     count, FFN1 1,083 -> 1,057, FFN2 887 -> 842, O-projection 325 -> 318,
//     and at most 1 % on normal data: the power limit takes it back.
//   - Fragment reads without bank conflicts (swz16).  With the swizzle of
//     32-row reads 44 % of the LDS's busy cycles were conflicts, FFN2 of
//     24,000 rows (N = 1024, K = 4096) took 180 us and not 169, QKV, FFN1 and
//     FFN2 of 262,144 rows 1 to 1.5 % more.
#include <algorithm>

#include "linear_common.h"

namespace surge {
namespace {

__device__ __forceinline__ bf16x8 lds_fragment(uint32_t addr) {
  return __builtin_bit_cast(bf16x8, *(const __attribute__((address_space(3))) u32x4*)addr);
}

// WAVES_M x WAVES_N waves of 16 (J0 + J1) tokens x 16 TI features; phase 0
// takes J0 of a wave's token fragments, phase 1 the other J1.
template <int WAVES_M, int WAVES_N, int TI, int J0, int J1, int EPI, int ORDER>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void linear_wide_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ W, const float* __restrict__ bias,
    const uint16_t* __restrict__ R, uint16_t* __restrict__ Y, int M, int N, int K, int tiles_n,
    int n_tiles, LinearExtra ex) {
  constexpr int TJ = J0 + J1;
  constexpr int R0 = 16 * J0, R1 = 16 * J1;  // a wave's token rows of either phase
  constexpr int BM = WAVES_M * (R0 + R1), BN = 256;
  constexpr int C1 = WAVES_M * R1 / 64;      // copies per wave of the phase-1 rows
  constexpr int CPS = 6 + C1;                // ... of a stage: 4 W, 2 phase-0 rows, C1
  static_assert(WAVES_M * WAVES_N == 8 && WAVES_N * TI == 16 && WAVES_M * R0 == 128 &&
                    WAVES_M * R1 == 64 * C1 && C1 <= 2 && J1 == 2 && TI * J0 == 16,
                "tiles of this kernel");
  // LDS, in bytes from smem: a stage of parity p at p * BUF, its W rows, then
  // (X0 on) its phase-0 and (X1 on) phase-1 rows of X, wave_m by wave_m; the
  // spare parts of the epilogue regions, 32 rows less the 8 C1 in copy slots.
  constexpr uint32_t X0 = 32768, X1 = X0 + 16384, BUF = X1 + C1 * 8192, SPARE = 2 * BUF;
  constexpr int SPARE_ROWS = 32 - 8 * C1;
  constexpr bool FOLD = EPI == EPI_FOLD || EPI == EPI_FOLD_GELU;
  constexpr bool LNRES = EPI == EPI_LNRES_STATS;
  constexpr int NV = 1 + (FOLD ? 1 : 0) + (LNRES ? 2 : 0);
  __shared__ __attribute__((aligned(128))) u32x4 smem[SPARE / 16 + 8 * SPARE_ROWS * 8];
  // Per-feature vectors (bias, then col_s or gamma and beta) by tile parity.
  __shared__ float4 svec[2][NV][BN / 4];
  __shared__ float2 srow[2][FOLD || LNRES ? 256 : 1];  // LayerNorm factors of the tile's rows

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave_m = wave / WAVES_N;
  const int wn0 = (wave % WAVES_N) * (16 * TI);
  const int wm0 = wave_m * (R0 + R1);
  const int nkt = K / 64;
  const int G = gridDim.x;

  // Fragment addresses: row lane % 16, then the swizzled 16-byte chunk of the
  // 32-wide K step ks, which for ks = 1 differs in bit 6 of the address only
  // (rows are 128 bytes, aligned); fragments are 16 rows apart.
  const uint32_t lds = lds_address(smem);
  uint32_t aw, ax, ax1;
  bf16x8 fw[TI][2], f0[J0][2], f1[J1][2];
  auto read_w = [&](int i, int ks) { fw[i][ks] = lds_fragment((aw ^ ks * 64) + i * 2048); };
  auto read_x0 = [&](int j, int ks) { f0[j][ks] = lds_fragment((ax ^ ks * 64) + j * 2048); };
  auto read_x1 = [&](int j, int ks) {  // (J0 == J1: the same rows, X1 - X0 on)
    f1[j][ks] = lds_fragment(((J0 == J1 ? ax + (X1 - X0) : ax1) ^ ks * 64) + j * 2048);
  };

  // Copies.  A wave instruction fills 8 rows of 128 bytes.
  const uint32_t ldsw = __builtin_amdgcn_readfirstlane(lds + wave * 1024);
  int it_tile = blockIdx.x;  // the copy stream's tile and stage
  int it_kt = 0;
  const uint16_t* xs;
  const uint16_t* ws;
  uint32_t xo[2 + C1];
  uint32_t wo;
  // A copy of the lane index that the compiler cannot see through: what is
  // derived from it is computed where it is used and not kept in registers
  // over the main loop, which has none to spare.
  auto opaque_lane = [&]() {
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  };
  // The addresses that stay the same over a tile but for the stage parity p;
  // formed at its start so that they take no registers over the epilogue.
  // With one register too many the allocator spilled wo, and the compiler
  // then waited for every copy in flight where it was used again, in each
  // K stage.
  auto tile_addresses = [&](uint32_t p) {
    const int l = opaque_lane();
    const uint32_t ch = (uint32_t)swz16(l & 15, l >> 4) * 16u + p * BUF;
    aw = lds + (uint32_t)wn0 * 128u + ch;
    ax = lds + X0 + (uint32_t)(wave_m * R0) * 128u + ch;
    ax1 = lds + X1 + (uint32_t)(wave_m * R1) * 128u + ch;
    wo = __umul24((uint32_t)(wave * 8 + (l >> 3)), (uint32_t)K * 2u) +
         (uint32_t)copy_chunk16(l) * 16u;
  };
  auto point = [&]() {
    int tm_, tn_;
    tile_coords<ORDER>(it_tile, n_tiles, tiles_n, &tm_, &tn_);
    xs = X + (size_t)(tm_ * BM) * K;
    ws = W + (size_t)(tn_ * BN) * K;
    const int l = opaque_lane();
#pragma unroll
    for (int q = 0; q < 2 + C1; ++q) {  // copies 0, 1: phase 0; rows past M: clamped
      const int lr = (q & 1) * 64 + wave * 8 + (l >> 3);
      const int row = q < 2 ? lr / R0 * (R0 + R1) + lr % R0 : lr / R1 * (R0 + R1) + R0 + lr % R1;
      xo[q] = __umul24((uint32_t)min(row, M - 1 - tm_ * BM), (uint32_t)K * 2u) +
              (uint32_t)copy_chunk16(l) * 16u;
    }
  };
  // Copy c of the cursor's stage into parity p, skipped where `go` is 0:
  // 0 .. 3 W, 4 .. 5 the phase-0 rows, 6 on the phase-1 rows.
  auto copy = [&](int c, uint32_t p, uint32_t go) {
    const uint32_t base = ldsw + p * BUF;
    if (c < 4)
      copy_to_lds16_if(ws + (size_t)(c * 64) * K + it_kt * 64, wo, base + c * 8192, go);
    else
      copy_to_lds16_if(xs + it_kt * 64, xo[c - 4], base + X0 + (c - 4) * 8192, go);
  };
  auto advance = [&]() {
    if (++it_kt == nkt) {
      it_kt = 0;
      it_tile += G;
      if (it_tile < n_tiles) point();
    }
  };
  auto more = [&]() { return lane_mask(it_tile < n_tiles); };

  int t = blockIdx.x;  // < n_tiles: the grid is never larger than the tile count
  point();
  tile_addresses(0);
  // Without row factors the launch has one tile per workgroup: thread r
  // merges the statistics of row r, before the first copy (a wait for the
  // loads is then no wait for copies).
  if constexpr (FOLD || LNRES) {
    if (!ex.rows_in && threadIdx.x < BM) {
      int tm, tn;
      tile_coords<ORDER>(t, n_tiles, tiles_n, &tm, &tn);
      const int m = min(tm * BM + (int)threadIdx.x, M - 1);
      srow[0][threadIdx.x] = ln_row_factors<RING_MAX_PARTS>(
          [&](int q) { return ex.stats_in[(size_t)q * M + m]; }, ex.parts_in, ex.eps);
    }
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const uint32_t go = more();
#pragma unroll
    for (int c = 0; c < CPS; ++c) copy(c, s, go);
    if (s == 0 || go) advance();
  }
  if (more())
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CPS) : "memory");
  else
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  uint32_t p = 0;  // parity of the stage being computed
  int tpar = 0;
  bool first = true;

  for (;;) {
    int tm, tn;
    tile_coords<ORDER>(t, n_tiles, tiles_n, &tm, &tn);
    const int m0 = tm * BM;
    const int n0 = tn * BN;
    tile_addresses(p);

    // Per-feature vectors, wave w copying vector w, and the row factors;
    // published by the barriers of the tile's first stages, last read two
    // tiles ago.
    if (wave < NV) {
      const float* src = bias;
      if constexpr (FOLD) { if (wave == 1) src = ex.col_s; }
      if constexpr (LNRES) { if (wave == 1) src = ex.gamma; if (wave == 2) src = ex.beta; }
      copy_lanes_to_lds16(src + n0, lds_address(&svec[tpar][wave][0]));
    }
    if constexpr (FOLD || LNRES) {  // 32 rows per wave
      const int l = opaque_lane();
      if (ex.rows_in)
        copy_to_lds4_at(ex.rows_in + m0,
                        (uint32_t)min(wave * 32 + (l >> 1), M - 1 - m0) * 8u + (uint32_t)(l & 1) * 4u,
                        lds_address(&srow[tpar][wave * 32]));
    }

    Acc acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) acc[i][j] = Acc{0.0f, 0.0f, 0.0f, 0.0f};

    // The tile's first stage: its W and phase-0 rows landed before the last
    // barrier A.
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int j = 0; j < J0; ++j) read_x0(j, ks);
#pragma unroll
      for (int i = 0; i < TI; ++i) read_w(i, ks);
    }

    for (int kt = 0; kt < nkt; ++kt) {
      const bool last = kt == nkt - 1;
      const uint32_t go = more();
      // Phase 0: 16 steps of two MFMAs.
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int ks = q >> 3, i = (q & 7) * 2 / J0, j = (q & 7) * 2 % J0;
        acc[i][j] = mma(fw[i][ks], f0[j][ks], acc[i][j]);
        acc[i][j + 1] = mma(fw[i][ks], f0[j + 1][ks], acc[i][j + 1]);
        if (q == 3) {
          // Barrier B: the phase-1 rows of this stage have landed (at a
          // tile's first stage they had before the previous epilogue's first
          // store); W and the phase-0 rows are read out.  CPS copies, or
          // more, were issued after those waited for, unless the stream has
          // ended.
          if (kt > 0) {
            if (go)
              asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CPS) : "memory");
            else
              asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          }
          __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
          __syncthreads();
        }
        if (q >= 4 && q < 8) read_x1(q & 1, (q - 4) >> 1);
        if (q >= 5 && (q & 1)) copy((q - 5) >> 1, p, go);
        __builtin_amdgcn_sched_barrier(0);
      }
      // Barrier A: W and the phase-0 rows of the next stage have landed (at a
      // tile's first stage as above); the phase-1 rows are read out.  (A tile
      // of one stage publishes its per-feature vectors here.)
      if (kt > 0 || first || nkt == 1) {
        if (go && nkt > 1)
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CPS) : "memory");
        else
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      __syncthreads();
      // The next stage is read from the other parity.
      const uint32_t other = p ? 0u - BUF : BUF;
      aw += other;
      ax += other;
      ax1 += other;
      const uint32_t go1 = lane_mask(go && !last);
      __builtin_amdgcn_sched_barrier(0);
      // Phase 1 (the fragments read at a tile's last stage are not used):
      // 2 TI steps of two MFMAs; the 2 J0 phase-0 fragments of the next stage
      // over the last steps.
#pragma unroll
      for (int q = 0; q < 2 * TI; ++q) {
        const int ks = q / TI, i = q % TI;
        acc[i][J0] = mma(fw[i][ks], f1[0][ks], acc[i][J0]);
        acc[i][J0 + 1] = mma(fw[i][ks], f1[1][ks], acc[i][J0 + 1]);
        read_w(i, ks);
        if (i >= TI - J0) read_x0(i - (TI - J0), ks);
        if ((q & 1) && q / 2 < C1) copy(6 + q / 2, p, go1);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (go1) advance();
      p ^= 1;
    }
    first = false;

    // The first region rows beside the stages, the last 8 C1 in this wave's
    // copy slots of the phase-1 rows of the last stage's parity.
    u32x4* const spare = smem + SPARE / 16 + wave * (SPARE_ROWS * 8);
    u32x4* const slots = smem + ((p ^ 1) * BUF + X1) / 16 + wave * 64;
    auto slot16 = [&](int r, int c) -> u32x4* {
      if (r < SPARE_ROWS) return spare + r * 8 + c;
      return slots + (r - SPARE_ROWS >= 8 ? 512 : 0) + (r & 7) * 8 + c;
    };
    auto vec = [&](int v, int q) { return svec[tpar][v][(wn0 >> 2) + q]; };
    auto rows = [&](int r) {
      if constexpr (FOLD || LNRES) return srow[tpar][wm0 + r];
      return float2{0.0f, 0.0f};
    };
    store_tile<TJ, TI, EPI>(acc, slot16, vec, rows, R, Y, m0 + wm0, n0 + wn0, M, N, opaque_lane(), ex);

    // The held-back copies, into slots only this wave has used since.
    const uint32_t go = more();
#pragma unroll
    for (int c = 6; c < CPS; ++c) copy(c, p ^ 1, go);
    if (go) advance();
    tpar ^= 1;
    t += G;
    if (t >= n_tiles) break;
  }
}

template <int BM, int WAVES_M, int WAVES_N, int TI, int J0>
hipError_t launch_wide_tiles(const uint16_t* X, const uint16_t* W, const float* bias,
                             const uint16_t* R, uint16_t* Y, int64_t M, int N, int K, int epi,
                             const LinearExtra& ex, hipStream_t stream) {
  const int tiles_n = N / 256;
  const int64_t n_tiles = (M + BM - 1) / BM * tiles_n;
  const bool factors = epi == EPI_FOLD || epi == EPI_FOLD_GELU || epi == EPI_LNRES_STATS;
  if (factors && !ex.rows_in && (ex.parts_in > RING_MAX_PARTS || n_tiles > ex.n_cus))
    return hipErrorInvalidValue;
  if (2 * K >= 1 << 24) return hipErrorInvalidValue;  // copy offsets: 24-bit row strides
  const dim3 grid((unsigned)std::min<int64_t>(n_tiles, ex.n_cus)), block(512);
#define SURGE_LAUNCH_EPI(E, O)                                                                 \
  hipLaunchKernelGGL((linear_wide_kernel<WAVES_M, WAVES_N, TI, J0, 2, E, O>), grid, block, 0, \
                     stream, X, W, bias, R, Y, (int)M, N, K, tiles_n, (int)n_tiles, ex)
  switch (epi) {
    case EPI_BIAS: SURGE_LAUNCH_EPI(EPI_BIAS, ORDER_ROW_GROUPS); break;
    case EPI_BIAS_GELU: SURGE_LAUNCH_EPI(EPI_BIAS_GELU, ORDER_FEATURE_HALVES); break;
    case EPI_BIAS_RESIDUAL: SURGE_LAUNCH_EPI(EPI_BIAS_RESIDUAL, ORDER_ROW_GROUPS); break;
    case EPI_FOLD: SURGE_LAUNCH_EPI(EPI_FOLD, ORDER_ROW_GROUPS); break;
    case EPI_FOLD_GELU: SURGE_LAUNCH_EPI(EPI_FOLD_GELU, ORDER_FEATURE_HALVES); break;
    case EPI_RES_STATS: SURGE_LAUNCH_EPI(EPI_RES_STATS, ORDER_ROW_GROUPS); break;
    default: SURGE_LAUNCH_EPI(EPI_LNRES_STATS, ORDER_ROW_GROUPS); break;
  }
#undef SURGE_LAUNCH_EPI
  return hipGetLastError();
}

}  // namespace

hipError_t launch_linear_wide(int rows, const uint16_t* X, const uint16_t* W, const float* bias,
                              const uint16_t* R, uint16_t* Y, int64_t M, int N, int K, int epi,
                              const LinearExtra& ex, hipStream_t stream) {
  if (rows == 192) return launch_wide_tiles<192, 2, 4, 4, 4>(X, W, bias, R, Y, M, N, K, epi, ex, stream);
  return launch_wide_tiles<256, 4, 2, 8, 2>(X, W, bias, R, Y, M, N, K, epi, ex, stream);
}

}  // namespace surge
