// Linear layers of small token counts (gfx950): Y = epi(X W^T + b) with few
// output tiles, where the time is one tile's chain of latencies and the
// stream of W through the few compute units that work.
//
// One workgroup computes one BM x BN tile (tokens x features) and ends.  K
// is walked in 128-wide stages through a ring of NBUF LDS buffers filled by
// direct global -> LDS copies: NBUF stages are in flight before the first
// MFMA, so the tile waits for memory latency about once and not once per
// stage.  Fragments of stage s + 1 are read while stage s is on the MFMA
// units; one barrier per stage publishes the next buffer and frees the
// current one.
//
// 32x32x16 MFMAs: half as many instructions on the tile's chain as the large
// tiles' 16x16x32 (one bge query 364 against 405 us), the same bits, and
// power does not count here.  The same K order, 64-feature statistics
// partials (summed in the same order) and finish too: a row's result does
// not depend on which kernel computed it.
//
// LayerNorm factors can come straight from the statistics partials of the
// producing layer (ex.stats_in): each tile merges its own rows' partials, so
// that no row-factor kernel runs between two layers.
#include "linear_common.h"

namespace surge {
namespace {

// Wait until at most `later` (<= MAXL) stages' copies (CPS instructions
// each) are still in flight; the vector memory counter retires in order.
template <int CPS, int MAXL>
__device__ __forceinline__ void wait_stages(int later) {
  if constexpr (MAXL <= 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    static_assert(CPS * MAXL <= 63, "vmcnt counts to 63");
    if (later >= MAXL)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CPS * MAXL) : "memory");
    else
      wait_stages<CPS, MAXL - 1>(later);
  }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int NBUF, int EPI>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64) void linear_ring_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ W, const float* __restrict__ bias,
    const uint16_t* __restrict__ R, uint16_t* __restrict__ Y, int M, int N, int K, int tiles_m,
    int tiles_n, LinearExtra ex) {
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int TM = BM / WAVES_M / 32;  // 32-token accumulator tiles per wave
  constexpr int TN = BN / WAVES_N / 32;  // 32-feature accumulator tiles per wave
  constexpr int CPR = 8;                 // 16-byte chunks per 64-wide LDS row
  constexpr int XI = BM / (8 * NW);      // copy instructions per wave per stage, X rows
  constexpr int WI = BN / (8 * NW);      // ... W rows
  constexpr int CPS = 2 * (XI + WI);      // ... a stage is two 64-wide halves
  constexpr int HALF = (BM + BN) * CPR;   // 16-byte slots of a half
  constexpr int STAGE = 2 * HALF;
  constexpr int PANELS = BN / STATS_WIDTH;
  constexpr bool FOLD = EPI == EPI_FOLD || EPI == EPI_FOLD_GELU;
  constexpr bool RES = EPI == EPI_BIAS_RESIDUAL || EPI == EPI_RES_STATS || EPI == EPI_LNRES_STATS;
  constexpr bool LNRES = EPI == EPI_LNRES_STATS;
  constexpr bool STATS = EPI == EPI_RES_STATS || EPI == EPI_LNRES_STATS;
  constexpr bool FACTORS = FOLD || LNRES;
  constexpr int NV = 1 + (FOLD ? 1 : 0) + (LNRES ? 2 : 0);
  static_assert(NW % 2 == 0 && XI >= 1 && WI >= 1, "copy slot phase needs an even wave count");
  static_assert(BN % STATS_WIDTH == 0 && TN <= 2 && BM <= 64, "tile shapes of this kernel");
  static_assert(TN == 2 || WAVES_N % 2 == 0, "a statistics partial is one wave or a wave pair");

  // A half of a stage: X rows, then W rows.  sT: the residual tile, overwritten in
  // place by the output tile, as PANELS panels of BM rows x 64 features.
  __shared__ u32x4 smem[NBUF * STAGE];
  __shared__ u32x4 sT[BN * BM / 8];
  __shared__ float4 svec[NV][BN / 4];
  __shared__ float2 spart[FACTORS ? RING_MAX_PARTS * BM : 1];
  __shared__ float4 sxch[STATS && TN == 1 ? (WAVES_N / 2) * BM * 2 : 1];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31;
  const int lhi = lane >> 5;
  const int wave_n = wave % WAVES_N;
  const int wn0 = wave_n * (BN / WAVES_N);
  const int wm0 = (wave / WAVES_N) * (BM / WAVES_M);
  const int nkt = K / 64;

  // Workgroups go round-robin over the 8 XCDs: each XCD takes a contiguous
  // run of tiles, walked along the token rows inside a feature block, so W
  // is split over the XCDs' L2s and read by one of them.
  int t = blockIdx.x;
  {
    const int n_tiles = tiles_m * tiles_n;
    const int per_xcd = n_tiles >> 3;
    if (t < per_xcd * 8) t = (t & 7) * per_xcd + (t >> 3);
  }
  const int m0 = (t % tiles_m) * BM;
  const int n0 = (t / tiles_m) * BN;

  const int dch = copy_chunk<CPR>(lane, wave);
  const int drow = wave * 8 + (lane >> 3);
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem) + wave * 1024);
  const uint16_t* xs = X + (size_t)m0 * K;
  const uint16_t* ws = W + (size_t)n0 * K;
  uint32_t xo[XI], wo[WI];
#pragma unroll
  for (int j = 0; j < XI; ++j)  // rows past M: clamped, never stored
    xo[j] = (uint32_t)(min(drow + j * NW * 8, M - 1 - m0) * K + dch * 8) * 2u;
#pragma unroll
  for (int j = 0; j < WI; ++j) wo[j] = (uint32_t)((drow + j * NW * 8) * K + dch * 8) * 2u;
  // An odd number of halves is made even by copying the last one twice.
  auto issue = [&](int st, int b) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int ko = min(2 * st + h, nkt - 1) * 64;
      const uint32_t base = lds0 + (uint32_t)(b * STAGE + h * HALF) * 16u;
#pragma unroll
      for (int j = 0; j < XI; ++j) copy_to_lds16_at(xs + ko, xo[j], base + j * NW * 1024);
#pragma unroll
      for (int j = 0; j < WI; ++j)
        copy_to_lds16_at(ws + ko, wo[j], base + BM * CPR * 16 + j * NW * 1024);
    }
  };

  // The epilogue's inputs first (they retire before stage 0): per-feature
  // vectors, the residual tile, and this tile's row factors or partials.
  if (wave == 0 && lane < BN / 4) {
    copy_lanes_to_lds16(bias + n0, lds_address(&svec[0][0]));
    if constexpr (FOLD) copy_lanes_to_lds16(ex.col_s + n0, lds_address(&svec[1][0]));
    if constexpr (LNRES) {
      copy_lanes_to_lds16(ex.gamma + n0, lds_address(&svec[1][0]));
      copy_lanes_to_lds16(ex.beta + n0, lds_address(&svec[2][0]));
    }
  }
  if constexpr (RES) {
    constexpr int RI = BM * PANELS / (8 * NW);  // 8-row copies per wave
#pragma unroll
    for (int j = 0; j < RI; ++j) {
      const int cidx = j * NW + wave;  // 8-row group: panel cidx / (BM/8)
      const int r = (cidx % (BM / 8)) * 8 + (lane >> 3);
      const int col = n0 + (cidx / (BM / 8)) * 64 + copy_chunk<CPR>(lane, cidx) * 8;
      copy_to_lds16(R + (size_t)min(m0 + r, M - 1) * N + col, lds_address(sT) + cidx * 1024);
    }
  }
  const int parts = FACTORS ? (ex.rows_in ? 1 : ex.parts_in) : 0;
  if constexpr (FACTORS) {
    const float2* src = ex.rows_in ? ex.rows_in : ex.stats_in;
    for (int p = wave; p < parts; p += NW)
#pragma unroll
      for (int h = 0; h < BM / 32; ++h)  // 32 rows x 8 bytes, 4 bytes per lane
        copy_to_lds4(reinterpret_cast<const float*>(
                         src + (size_t)p * M + min(m0 + h * 32 + (lane >> 1), M - 1)) + (lane & 1),
                     lds_address(spart) + (uint32_t)(p * BM + h * 32) * 8u);
  }

  const int ns = (nkt + 1) >> 1;  // stages
#pragma unroll
  for (int b = 0; b < NBUF; ++b)
    if (b < ns) issue(b, b);

  f32x16 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  bf16x8 fa[2][8][TN], fb[2][8][TM];
  auto read = [&](int b, int set) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const u32x4* sx = smem + b * STAGE + (ks >> 2) * HALF;
      const u32x4* sw = sx + BM * CPR;
      const int ch = (ks & 3) * 2 + lhi;
#pragma unroll
      for (int i = 0; i < TN; ++i)
        fa[set][ks][i] = __builtin_bit_cast(bf16x8, sw[swz<CPR>(wn0 + i * 32 + l32, ch)]);
#pragma unroll
      for (int j = 0; j < TM; ++j)
        fb[set][ks][j] = __builtin_bit_cast(bf16x8, sx[swz<CPR>(wm0 + j * 32 + l32, ch)]);
    }
  };
  auto multiply = [&](int set, int from, int to) {
#pragma unroll
    for (int ks = from; ks < to; ++ks)
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][ks][i], fb[set][ks][j],
                                                              acc[i][j], 0, 0, 0);
  };
  // This wave's fragment reads are done (a form the compiler counts too).
  auto reads_done = [] { __builtin_amdgcn_s_waitcnt(0xC07F); };  // lgkmcnt(0)

  wait_stages<CPS, NBUF - 1>(ns - 1);
  __syncthreads();
  read(0, 0);

  // Before stage s runs on the MFMA units: stage s + 1 has landed and every
  // wave has read stage s, so its buffer nb takes stage s + NBUF.
  int nb = 0;
  auto refill = [&](int s, int set) {
    reads_done();
    __syncthreads();
    issue(s + NBUF, nb);
    nb = nb + 1 == NBUF ? 0 : nb + 1;
    read(nb, set ^ 1);
    multiply(set, 0, 8);
  };
  auto drain = [&](int s, int set) {
    wait_stages<CPS, NBUF - 2>(ns - 2 - s);
    reads_done();
    __syncthreads();
    nb = nb + 1 == NBUF ? 0 : nb + 1;
    read(nb, set ^ 1);
    multiply(set, 0, 8);
  };
  int s = 0;
  for (; s + NBUF + 1 < ns; s += 2) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CPS * (NBUF - 2)) : "memory");
    refill(s, 0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CPS * (NBUF - 2)) : "memory");
    refill(s + 1, 1);
  }
  // At most NBUF + 1 stages are left, the last of them perhaps a half.
  if (s + NBUF < ns) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(CPS * (NBUF - 2)) : "memory");
    refill(s, 0);
    ++s;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {  // the sets change places
#pragma unroll
      for (int i = 0; i < TN; ++i) fa[0][ks][i] = fa[1][ks][i];
#pragma unroll
      for (int j = 0; j < TM; ++j) fb[0][ks][j] = fb[1][ks][j];
    }
  }
  for (; s + 2 < ns; s += 2) {
    drain(s, 0);
    drain(s + 1, 1);
  }
  const bool whole = (nkt & 1) == 0;
  if (s + 1 < ns) {
    drain(s, 0);
    reads_done();
    multiply(1, 0, 4);
    if (whole) multiply(1, 4, 8);
  } else {
    reads_done();
    multiply(0, 0, 4);
    if (whole) multiply(0, 4, 8);
  }

  // acc[i][j] register r holds Y[m][n] with m = m0 + wm0 + j*32 + lane%32,
  // n = n0 + wn0 + i*32 + 8*(r/4) + 4*(lane/32) + r%4.
  float rs[TM], nm[TM];
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    rs[j] = nm[j] = 0.0f;
    if constexpr (FACTORS) {
      const int row = wm0 + j * 32 + l32;
      if (ex.rows_in) {
        rs[j] = spart[row].x;
        nm[j] = spart[row].y;
      } else {
        const float2 f = ln_row_factors<RING_MAX_PARTS>([&](int p) { return spart[p * BM + row]; },
                                                        parts, ex.eps);
        rs[j] = f.x;
        nm[j] = f.y;
      }
    }
  }
  uint2 out[TN][TM][4];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int row = wm0 + j * 32 + l32;
        const int f = wn0 + i * 32 + 8 * g + 4 * lhi;  // first of the 4 features, in the tile
        const float4 bb = svec[0][f >> 2];
        float4 cs = {0.0f, 0.0f, 0.0f, 0.0f}, gg = cs, be = cs;
        if constexpr (FOLD) cs = svec[1][f >> 2];
        if constexpr (LNRES) {
          gg = svec[1][f >> 2];
          be = svec[2][f >> 2];
        }
        uint2* cell = reinterpret_cast<uint2*>(
                          &sT[(f >> 6) * BM * CPR + swz<CPR>(row, (f & 63) >> 3)]) + lhi;
        const float a[4] = {acc[i][j][4 * g + 0], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2],
                            acc[i][j][4 * g + 3]};
        uint2 res = {0u, 0u};
        if constexpr (RES) res = *cell;
        out[i][j][g] = finish4<EPI>(a, bb, cs, gg, be, rs[j], nm[j], res);
        *cell = out[i][j][g];
      }

  // Row statistics over 64 features: one wave's two accumulator tiles, or
  // (TN = 1) a pair of waves, the second continuing the first's sums.  In
  // the 16x16x32 layout of the large tiles the four lanes of a token hold
  // features 4q .. 4q+3 of every 16; this lane holds those of q = lhi (even
  // g) and of q = 2 + lhi (odd g), summed apart to add up in the same order.
  if constexpr (STATS) {
    float ss[TM][2], sq[TM][2];
    auto add = [&](int i, int j) {
#pragma unroll
      for (int g = 0; g < 4; ++g) row_stats_add(out[i][j][g], ss[j][g & 1], sq[j][g & 1]);
    };
    auto finish = [&](int j) {
      float s2[2], q2[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        s2[h] = ss[j][h] + __shfl_xor(ss[j][h], 32, 64);
        q2[h] = sq[j][h] + __shfl_xor(sq[j][h], 32, 64);
      }
      const int m = m0 + wm0 + j * 32 + l32;
      if (lhi == 0 && m < M)
        ex.stats_out[(size_t)((n0 + wn0) / STATS_WIDTH) * M + m] =
            row_stats_finish(s2[0] + s2[1], q2[0] + q2[1]);
    };
#pragma unroll
    for (int j = 0; j < TM; ++j) ss[j][0] = ss[j][1] = sq[j][0] = sq[j][1] = 0.0f;
    if constexpr (TN == 2) {
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        add(0, j);
        add(1, j);
        finish(j);
      }
    } else {
      float4* x = sxch + (wave_n / 2) * BM * 2;
      if (wave_n % 2 == 0) {
#pragma unroll
        for (int j = 0; j < TM; ++j) {
          add(0, j);
          x[(wm0 + j * 32 + l32) * 2 + lhi] = make_float4(ss[j][0], ss[j][1], sq[j][0], sq[j][1]);
        }
      }
      __syncthreads();
      if (wave_n % 2 == 1) {
#pragma unroll
        for (int j = 0; j < TM; ++j) {
          const float4 v = x[(wm0 + j * 32 + l32) * 2 + lhi];
          ss[j][0] = v.x;
          ss[j][1] = v.y;
          sq[j][0] = v.z;
          sq[j][1] = v.w;
          add(0, j);
          finish(j);
        }
      }
    }
  }
  __syncthreads();

  // The output tile as whole 128-byte row segments.
#pragma unroll
  for (int j = 0; j < BM * PANELS / (8 * NW); ++j) {
    const int cidx = j * NW + wave;
    const int m = m0 + (cidx % (BM / 8)) * 8 + (lane >> 3);
    const int col = n0 + (cidx / (BM / 8)) * 64 + copy_chunk<CPR>(lane, cidx) * 8;
    const u32x4 v = sT[cidx * 64 + lane];
    if (m < M) *reinterpret_cast<u32x4*>(Y + (size_t)m * N + col) = v;
  }
}

}  // namespace

template <int BM, int BN, int WAVES_M, int WAVES_N, int NBUF>
hipError_t launch_ring_tiles(const uint16_t* X, const uint16_t* W, const float* bias,
                             const uint16_t* R, uint16_t* Y, int64_t M, int N, int K, int epi,
                             const LinearExtra& ex, hipStream_t stream) {
  if ((int64_t)BN * K * 2 > (int64_t)UINT32_MAX) return hipErrorInvalidValue;  // copy offsets
  const bool factors = epi == EPI_FOLD || epi == EPI_FOLD_GELU || epi == EPI_LNRES_STATS;
  if (factors && !ex.rows_in && ex.parts_in > RING_MAX_PARTS) return hipErrorInvalidValue;
  const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = N / BN;
  const dim3 grid((unsigned)(tiles_m * tiles_n)), block(WAVES_M * WAVES_N * 64);
#define SURGE_LAUNCH_EPI(E)                                                                     \
  hipLaunchKernelGGL((linear_ring_kernel<BM, BN, WAVES_M, WAVES_N, NBUF, E>), grid, block, 0, stream, \
                     X, W, bias, R, Y, (int)M, N, K, tiles_m, tiles_n, ex)
  switch (epi) {
    case EPI_BIAS: SURGE_LAUNCH_EPI(EPI_BIAS); break;
    case EPI_BIAS_GELU: SURGE_LAUNCH_EPI(EPI_BIAS_GELU); break;
    case EPI_BIAS_RESIDUAL: SURGE_LAUNCH_EPI(EPI_BIAS_RESIDUAL); break;
    case EPI_FOLD: SURGE_LAUNCH_EPI(EPI_FOLD); break;
    case EPI_FOLD_GELU: SURGE_LAUNCH_EPI(EPI_FOLD_GELU); break;
    case EPI_RES_STATS: SURGE_LAUNCH_EPI(EPI_RES_STATS); break;
    default: SURGE_LAUNCH_EPI(EPI_LNRES_STATS); break;
  }
#undef SURGE_LAUNCH_EPI
  return hipGetLastError();
}

hipError_t launch_linear_ring(RingTile tile, const uint16_t* X, const uint16_t* W,
                              const float* bias, const uint16_t* R, uint16_t* Y, int64_t M, int N,
                              int K, int epi, const LinearExtra& ex, hipStream_t stream) {
  switch (tile) {
    case RING_32x64:
      return launch_ring_tiles<32, 64, 1, 2, 3>(X, W, bias, R, Y, M, N, K, epi, ex, stream);
    case RING_64x64:
      return launch_ring_tiles<64, 64, 2, 2, 3>(X, W, bias, R, Y, M, N, K, epi, ex, stream);
    default:
      return launch_ring_tiles<64, 128, 2, 2, 2>(X, W, bias, R, Y, M, N, K, epi, ex, stream);
  }
}

}  // namespace surge
