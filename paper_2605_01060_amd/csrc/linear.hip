// Token-major linear layers on bf16 MFMA (gfx950): Y = epi(X W^T + b).
//
// X is the packed token matrix [M, K] (M = tokens of the chunk, no padding),
// W the layer weight repacked to [N, K] so both operands are K-contiguous.
//
// Three tile families share the operand layout, the K order and the finish
// of every output, and launch_linear picks one by the launch's tile counts:
// small chunks (linear_ring.hip), 256 x 256 or 192 x 256 tiles
// (linear_wide.hip), and the 128 x 128 tiles of this file in between and for
// the odd last 128 features of an N that is not a multiple of 256.
//
// Tiling.  A workgroup computes 128 x 128 tiles of Y (tokens x features) with
// four waves of 64 x 64 (16x16x32 bf16 MFMAs).  K is walked in 64-wide stages
// through a double-buffered LDS tile.
//
// Persistence.  The grid holds as many workgroups as fit on the chip at
// once; workgroup b computes tiles b, b + G, b + 2G, ... (G = grid size).
// The copy pipeline runs on across tile boundaries: the next tile's first
// stage is copied while the current tile's last stage is on the MFMA units,
// and its second stage as soon as each wave has finished its epilogue.  A
// tile therefore never starts on an empty pipeline, and no workgroup launch
// separates two tiles.
//
// Epilogue memory.  The buffer released by a tile's last stage is idle
// until the next tile's second stage is copied into it, so each wave uses
// the slots its own copies of that stage will fill as its 4 KB epilogue
// region, and issues those copies when its epilogue is done (no other wave
// touches the slots, so no barrier is needed).  The tile's per-feature
// vectors (bias, and the LayerNorm columns of the fused forms) are copied
// into LDS once per tile at its start, so the epilogue reads them from LDS
// instead of every lane fetching them again from global memory.  The
// output rows and the residual rows are touched once per launch, so they
// are stored and loaded nontemporally, leaving the L2 to the operand tiles
// that other workgroups read again.
//
// Staging.  Stage k+2 is copied straight from global memory into the LDS
// buffer stage k has just released (global_load_lds_dwordx4, 1 KB per wave
// instruction) while stage k+1 runs on the MFMA units; one wait and one
// barrier per stage.  An LDS row holds 64 bf16 of one X or W row as eight
// 16-byte chunks; the logical chunk c of row r is stored at position
// c ^ (r & 7), which leaves a fragment read (four logical chunks from 16
// consecutive rows, 16 lanes a chunk) free of bank conflicts.  A copy
// instruction writes 64 consecutive slots, so each lane fetches the logical
// chunk that belongs in its slot.
//
// Occupancy.  Two workgroups per CU (64 + 4 KB of LDS each), 2 waves per
// SIMD.
//
// Operand roles.  The MFMA A operand is the weight tile and B the token
// tile, so the accumulators hold Y^T: each lane owns one token row and four
// consecutive features per register group.
//
// Every output row is computed from its own input row with a fixed K order
// (no split-K, no atomics), so a text's result does not depend on which
// other texts share its SuperBatch or chunk, nor on the tile configuration.
#include <algorithm>

#include "linear_common.h"

namespace surge {
namespace {

// With MERGE the rows' LayerNorm factors come from the statistics partials
// (ex.stats_in): lane r of a wave loads those of the wave's row r at the
// tile's start, so that their latency hides behind the main loop, and merges
// them before the epilogue.  Otherwise the lane loads the row's factors.
template <int EPI, int ORDER, bool MERGE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void linear_bf16_kernel(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W,
                        const float* __restrict__ bias, const uint16_t* __restrict__ R,
                        uint16_t* __restrict__ Y, int M, int N, int K, int tiles_n, int n_tiles,
                        LinearExtra ex) {
  constexpr int BM = 128, BN = 128, BK = 64;
  constexpr int NWAVES = 4, WAVES_N = 2;
  constexpr int WM = 64, WN = 64;   // tokens, features per wave
  constexpr int TI = WN / 16;       // 16-feature fragments per wave
  constexpr int TJ = WM / 16;       // 16-token fragments per wave
  constexpr int CPR = BK / 8;       // 16-byte chunks per LDS row
  constexpr int RPC = 64 / CPR;     // rows one wave copy instruction fills
  constexpr int XI = BM / (RPC * NWAVES);  // copy instructions per wave per stage, X tile
  constexpr int WI = BN / (RPC * NWAVES);  // ... W tile
  constexpr int SSTAGE = (BM + BN) * CPR;  // 16-byte slots per stage buffer
  // Buffer b holds X rows at smem[b*SSTAGE ..] and W rows after them.
  __shared__ u32x4 smem[2 * SSTAGE];
  // Per-feature vectors of the current tile (bias, then col_s or gamma and
  // beta), double-buffered by the parity of the workgroup's tile count.
  constexpr bool FOLD_ = EPI == EPI_FOLD || EPI == EPI_FOLD_GELU;
  constexpr bool LNRES_ = EPI == EPI_LNRES_STATS;
  constexpr int NV = 1 + (FOLD_ ? 1 : 0) + (LNRES_ ? 2 : 0);
  static_assert(NV <= NWAVES, "one vector per wave copy");
  __shared__ float4 svec[2][NV][BN / 4];
  static_assert(XI >= 4, "a wave's epilogue region is 4 of its X copy slots");

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: kept in an SGPR
  const int l16 = lane & 15;
  const int lq = lane >> 4;
  const int wn0 = (wave % WAVES_N) * WN;
  const int wm0 = (wave / WAVES_N) * WM;
  const int nkt = K / BK;
  const int G = gridDim.x;

  // Lane l of wave w, copy j, fills LDS slot p = (j*NWAVES + w)*64 + l of a
  // tile: row p / 8, stored chunk l % 8.  Its logical chunk
  // (l & 7) ^ (l >> 3) is the same for every j; its rows are NWAVES * 8
  // apart.
  constexpr int DSTEP = NWAVES * RPC;
  const int drow = wave * RPC + lane / CPR;
  const int dch = copy_chunk16(lane);
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem) + wave * 64 * 16);
  constexpr uint32_t STAGE_BYTES = SSTAGE * 16;
  constexpr uint32_t COPY_BYTES = NWAVES * 64 * 16;

  // The copy stream runs two stages ahead of the MFMA work through this
  // workgroup's sequence of (tile, stage) pairs.  The issue cursor holds
  // the tile and stage to copy next and the source pointers of that tile;
  // advancing past a tile's last stage moves it to the workgroup's next
  // tile (that work stays off the path between a barrier and the MFMAs).
  int it_tile = blockIdx.x;  // < n_tiles: the grid is never larger than the tile count
  int it_kt = 0;
  // Copy sources: a wave-uniform tile base (scalar registers) plus a 32-bit
  // byte offset per lane that stays fixed while the tile's stages advance,
  // so a copy needs no per-lane address arithmetic (the launcher checks that
  // BM rows of K bf16 fit the 32-bit offset).
  const uint16_t* xs;  // X row block of the tile
  const uint16_t* ws;  // W feature block of the tile
  uint32_t xo[XI], wo[WI];
#pragma unroll
  for (int j = 0; j < WI; ++j) wo[j] = (uint32_t)((drow + j * DSTEP) * K + dch * 8) * 2u;
  auto point = [&]() {
    int tm_, tn_;
    tile_coords<ORDER>(it_tile, n_tiles, tiles_n, &tm_, &tn_);
    xs = X + (size_t)(tm_ * BM) * K;
    ws = W + (size_t)(tn_ * BN) * K;
#pragma unroll
    for (int j = 0; j < XI; ++j)  // rows past M: clamped, never stored
      xo[j] = (uint32_t)((min(tm_ * BM + drow + j * DSTEP, M - 1) - tm_ * BM) * K + dch * 8) * 2u;
  };
  auto issue = [&](int b) {
    if (it_tile >= n_tiles) return;
    const int ko = it_kt * BK;
    const uint32_t base = lds0 + (uint32_t)b * STAGE_BYTES;
    const uint16_t* sx = xs + ko;
    const uint16_t* sw = ws + ko;
#pragma unroll
    for (int j = 0; j < XI; ++j) copy_to_lds16_at(sx, xo[j], base + j * COPY_BYTES);
#pragma unroll
    for (int j = 0; j < WI; ++j) copy_to_lds16_at(sw, wo[j], base + BM * CPR * 16 + j * COPY_BYTES);
  };
  auto advance = [&]() {
    if (++it_kt == nkt) {
      it_kt = 0;
      it_tile += G;
      if (it_tile < n_tiles) point();
    }
  };

  int t = blockIdx.x;
  point();
  issue(0);
  advance();
  const bool second = it_tile < n_tiles;
  issue(1);
  advance();
  if (second)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(XI + WI) : "memory");
  else
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  constexpr int S = BK / 32;   // 32-wide MFMA steps per stage
  constexpr int NR = TI + TJ;  // fragment reads per step
  constexpr int NM = TI * TJ;  // MFMAs per step
  static_assert(S == 2, "fragment parity must restart at every stage");
  static_assert(NM >= NR, "interleave needs at least one MFMA per read");
  bf16x8 fa[2][TI], fb[2][TJ];
  // Fragments of K step ks of a stage buffer, and a step's MFMAs.
  auto read = [&](const u32x4* sx, int ks) {
    const u32x4* sw = sx + BM * CPR;
#pragma unroll
    for (int i = 0; i < TI; ++i)
      fa[ks][i] = __builtin_bit_cast(bf16x8, sw[swz16(wn0 + i * 16 + l16, ks * 4 + lq)]);
#pragma unroll
    for (int j = 0; j < TJ; ++j)
      fb[ks][j] = __builtin_bit_cast(bf16x8, sx[swz16(wm0 + j * 16 + l16, ks * 4 + lq)]);
  };
  int cur_buf = 0;
  int tpar = 0;

  for (;;) {
    int tm, tn;
    tile_coords<ORDER>(t, n_tiles, tiles_n, &tm, &tn);
    const int m0 = tm * BM;
    const int n0 = tn * BN;

    // This tile's per-feature vectors into svec[tpar], wave w copying
    // vector w (BN floats: one 16-byte chunk per lane).  The main loop's
    // first stage waits for every copy and meets at a barrier, so the
    // epilogue finds them in place; the buffer was last read by the
    // epilogue two tiles back.
    if (wave < NV && lane < BN / 4) {
      const float* src = bias;
      if constexpr (FOLD_) { if (wave == 1) src = ex.col_s; }
      if constexpr (LNRES_) { if (wave == 1) src = ex.gamma; if (wave == 2) src = ex.beta; }
      copy_lanes_to_lds16(src + n0, lds_address(&svec[tpar][wave][0]));
    }

    // LayerNorm factors of the wave's row `lane` (fused LayerNorm epilogues).
    constexpr int MAXP = MERGE ? RING_MAX_PARTS : 1;
    float2 rowf[MAXP];
    if constexpr (FOLD_ || LNRES_) {
      const int m = min(m0 + wm0 + lane, M - 1);
      if constexpr (MERGE) {
#pragma unroll
        for (int q = 0; q < MAXP; ++q)
          if (q < ex.parts_in) rowf[q] = ex.stats_in[(size_t)q * M + m];
      } else {
        rowf[0] = ex.rows_in[m];
      }
    }

    Acc acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) acc[i][j] = Acc{0.0f, 0.0f, 0.0f, 0.0f};
    auto step = [&](int ks) {
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = mma(fa[ks][i], fb[ks][j], acc[i][j]);
      // Pin: the MFMAs above with the fragment reads around them one by one.
#pragma unroll
      for (int x = 0; x < NR; ++x) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // LDS read
      }
      __builtin_amdgcn_sched_group_barrier(0x008, NM - NR, 0);
    };

    read(smem + cur_buf * SSTAGE, 0);

    // One stage per trip.  The first step runs its MFMAs with the fragment
    // reads of the second interleaved one by one (pinned with scheduling
    // group barriers).  Then the wave waits for everything it issued before
    // (the copies of the next stage; at a tile's first stage also the
    // previous tile's epilogue loads and stores) and all waves meet: the next
    // stage is published and nobody reads this stage's buffer any more, so
    // the copies of the stage after next go into it.  The second step's
    // MFMAs, which need no LDS, run after the barrier while the first
    // fragments of the next stage are read, so the MFMA pipe does not wait
    // for LDS at the stage boundary.  (At a tile's last stage those reads are
    // discarded; the next tile reads its own after the epilogue.)
    for (int kt = 0; kt < nkt; ++kt) {
      read(smem + cur_buf * SSTAGE, 1);
      step(0);
      // None of these MFMAs behind the barrier, where the next copies would
      // wait for their issue: in launches of few tiles a stage is as long as
      // its copies take (N = 768, K = 3072, us: M = 4000 35.2 -> 33.5, 7000
      // 43.3 -> 40.7; N = 384, K = 1536, 265,000 rows 480 -> 468).
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this stage's reads are done
      __syncthreads();
      const bool last_stage = kt == nkt - 1;
      if (!last_stage) issue(cur_buf);
      cur_buf ^= 1;
      read(smem + cur_buf * SSTAGE, 0);
      step(1);
      if (!last_stage) advance();
    }

    // Region row r lives in this wave's X copy slot r/8 of the buffer the
    // last stage released (8 rows of 128 bytes per 1 KB slot).
    u32x4* const rbase = smem + (cur_buf ^ 1) * SSTAGE + wave * 64;
    auto slot16 = [&](int r, int c) -> u32x4* {
      return rbase + (r >> 3) * (NWAVES * 64) + (r & 7) * 8 + c;
    };
    auto vec = [&](int v, int q) { return svec[tpar][v][(wn0 >> 2) + q]; };
    float2 own = make_float2(0.0f, 0.0f);
    if constexpr (FOLD_ || LNRES_) {
      own = rowf[0];
      if constexpr (MERGE)
        own = ln_row_factors<MAXP>([&](int q) { return rowf[q]; }, ex.parts_in, ex.eps);
    }
    auto rows = [&](int r) {
      return make_float2(__shfl(own.x, r, 64), __shfl(own.y, r, 64));
    };
    store_tile<TJ, TI, EPI>(acc, slot16, vec, rows, R, Y, m0 + wm0, n0 + wn0, M, N, lane, ex);

    // The region's reads are done (waited above); this wave's deferred copies
    // of the next tile's second stage go into the same slots.
    issue(cur_buf ^ 1);
    advance();
    tpar ^= 1;
    t += G;
    if (t >= n_tiles) break;
  }
}

// The first `cols` of the N features.
hipError_t launch_mid(const uint16_t* X, const uint16_t* W, const float* bias, const uint16_t* R,
                      uint16_t* Y, int64_t M, int N, int cols, int K, int epi,
                      const LinearExtra& ex, hipStream_t stream) {
  constexpr int BM = 128, BN = 128, PER_CU = 2;
  if ((int64_t)BM * K * 2 > (int64_t)UINT32_MAX) return hipErrorInvalidValue;  // copy offsets
  const int tiles_n = cols / BN;
  const int64_t tiles_m = (M + BM - 1) / BM;
  const int n_tiles = (int)(tiles_m * tiles_n);
  const dim3 grid((unsigned)std::min<int64_t>(n_tiles, (int64_t)ex.n_cus * PER_CU));
  const dim3 block(256);
  // Only the epilogues with LayerNorm factors have a MERGE kernel.
#define SURGE_LAUNCH(E, O, MERGE)                                                               \
  hipLaunchKernelGGL((linear_bf16_kernel<E, O, MERGE>), grid, block, 0, stream, X, W, bias, R, Y, \
                     (int)M, N, K, tiles_n, n_tiles, ex)
#define SURGE_LAUNCH_FACTORS(E, O)   \
  if (ex.rows_in)                    \
    SURGE_LAUNCH(E, O, false);       \
  else                               \
    SURGE_LAUNCH(E, O, true)
  switch (epi) {
    case EPI_BIAS: SURGE_LAUNCH(EPI_BIAS, ORDER_ROW_GROUPS, false); break;
    case EPI_BIAS_GELU: SURGE_LAUNCH(EPI_BIAS_GELU, ORDER_FEATURE_HALVES, false); break;
    case EPI_BIAS_RESIDUAL: SURGE_LAUNCH(EPI_BIAS_RESIDUAL, ORDER_ROW_GROUPS, false); break;
    case EPI_FOLD: SURGE_LAUNCH_FACTORS(EPI_FOLD, ORDER_ROW_GROUPS); break;
    case EPI_FOLD_GELU: SURGE_LAUNCH_FACTORS(EPI_FOLD_GELU, ORDER_FEATURE_HALVES); break;
    case EPI_RES_STATS: SURGE_LAUNCH(EPI_RES_STATS, ORDER_ROW_GROUPS, false); break;
    default: SURGE_LAUNCH_FACTORS(EPI_LNRES_STATS, ORDER_ROW_GROUPS); break;
  }
#undef SURGE_LAUNCH_FACTORS
#undef SURGE_LAUNCH
  return hipGetLastError();
}

}  // namespace

// Small chunks, where a tile's own chain of latencies is the launch's time:
// the smallest tile of which there is still at most one per CU.  A smaller
// tile is a shorter chain (copies, barrier and MFMAs per stage) and spreads
// the stream of W over more CUs; once there is more than one per CU the
// shared operand traffic costs more than it saves.  Measured (us per layer,
// K = 3072, N = 768; 32x64 / 64x64 / 64x128 / 128x128 persistent tiles):
//   M = 24    7.8 / 9.9 / 15.7 / 24.2      M = 512   8.1 / 10.1 / 16.1 / 24.9
//   M = 1024  14.4 / 11.5 / 21.0 / 33.0    M = 2080  30.2 / 26.8 / 23.4 / 32.0
//   M = 4096  47.8 / 45.3 / 45.0 / 31.7.
static RingTile ring_tile(int64_t M, int N, int n_cus) {
  auto fits = [&](int bm, int bn) { return (M + bm - 1) / bm * (N / bn) <= n_cus; };
  if (fits(32, 64)) return RING_32x64;
  if (fits(64, 64)) return RING_64x64;
  if (fits(64, 128)) return RING_64x128;
  return RING_NONE;
}

int linear_stats_width(int64_t, int) { return STATS_WIDTH; }

hipError_t resolve_cus(int* n_cus) {
  if (*n_cus > 0) return hipSuccess;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  return hipDeviceGetAttribute(n_cus, hipDeviceAttributeMultiprocessorCount, dev);
}

// Which family a launch takes: beyond the small chunks 256 x 256 or 192 x 256
// tiles (one workgroup per CU) or 128 x 128 tiles (two), by the cost of their
// rounds.  The unit is a full round of 128-wide tiles.  Those fill the chip by
// halves of a round and end about 0.07 late; a round of 256-row tiles does
// twice the work in 1.4 + 240 / (K + 400) units (the less, the more main loop
// there is per epilogue: 1.45 at K = 4096, at most 1.85, where stores bound
// both), the first 50 / K later (copies with no main loop to hide behind), and
// one of 192-row tiles three quarters of that in 0.834 of the time (fewer
// MFMAs per operand byte), but a begun round costs a whole one.  Fitted to
// 1,814 launches of N = 256 .. 4096, K = 64 .. 4096, M = 2500 .. 262,144 timed
// under each family: the mean one takes 0.2 % longer than under its best, the
// worst 8 %.  Measured (us, 128 / 192 / 256 rows):
//   N = 2304, K = 768   M = 6144 28.2 / 35.5 / 23.9    8192 34.5 / 36.6 / 43.4
//                       10,000 42.3 / 39.2 / 44.6      13,579 56.0 / 56.0 / 49.8
//   N = 768, K = 3072   M = 8192 44.7 / 52.0 / 64.3    13,579 79.6 / 61.2 / 66.8
//                       17,000 89.7 / 114 / 77.5       262,144 1,299 / 1,096 / 1,026
//   N = 768, K = 256    M = 8192 7.9 / 9.6 / 11.4      262,144 149 / 140 / 131
//   N = 2304, K = 64    M = 13,579 16.9 / 19.8 / 19.1  262,144 235 / 235 / 226.
// An odd last 128 features take 128-wide tiles in a launch of their own, which
// reads X once more and costs 0.7 units beside its rounds.  1,058 launches of
// N = 384 .. 2432 are 0.2 % off their best in the mean (8 % at worst); all on
// 128-wide tiles they are 1.5 % (49 %).  Measured (us, 128 / 128 and 256): N =
// 1152, K = 64 M = 140,000 67.4 / 70.7, K = 3072 55,000 417 / 386; N = 640, K =
// 3072 20,781 89.2 / 109, 75,000 320 / 363; N = 896, K = 768 100,000 184 / 182.
// With one column of 256-wide tiles before them (N = 384) it never paid: K =
// 768 M = 262,144 199 / 213, K = 1536 100,000 150 / 177.
enum Family { FAMILY_RING, FAMILY_MID, FAMILY_WIDE, FAMILY_WIDE_AND_MID };
struct Choice {
  Family family;
  int rows;  // of a tile, but for FAMILY_RING's
};
static Choice linear_family(int64_t M, int N, int K, int n_cus) {
  if (ring_tile(M, N, n_cus) != RING_NONE) return {FAMILY_RING, 0};
  // The wide tiles' copy offsets are products of 24-bit numbers.
  if (K >= 1 << 23) return {FAMILY_MID, 128};
  auto rounds = [&](int64_t bm, int columns) {
    return (double)(((M + bm - 1) / bm * columns + n_cus - 1) / n_cus);
  };
  auto mid = [&](int columns) { return 0.5 * rounds(128, columns) + 0.07; };
  const double wide = std::min(1.4 + 240.0 / (K + 400), 1.85);
  const double c256 = 50.0 / K + wide * rounds(256, N / 256);
  if (N % 256 != 0) {
    const bool split = N > 512 && c256 + mid(1) + 0.7 < mid(N / 128);
    return split ? Choice{FAMILY_WIDE_AND_MID, 256} : Choice{FAMILY_MID, 128};
  }
  const double c128 = mid(N / 128), c192 = 0.834 * wide * rounds(192, N / 256);
  if (c192 < c256 && c192 < c128) return {FAMILY_WIDE, 192};
  return c256 <= c128 ? Choice{FAMILY_WIDE, 256} : Choice{FAMILY_MID, 128};
}

int linear_tile(int64_t M, int N, int K, int n_cus) {
  const Choice c = linear_family(M, N, K, n_cus);
  if (c.family != FAMILY_RING) return c.rows << 16 | (c.family == FAMILY_MID ? 128 : 256);
  const RingTile t = ring_tile(M, N, n_cus);
  return (t == RING_32x64 ? 32 : 64) << 16 | (t == RING_64x128 ? 128 : 64);
}

// The tiles merge statistics where that costs less than a row-factor launch
// (5 us with its gap): always in small chunks; 128-wide tiles hide the loads
// but repeat them for every feature tile, up to four rounds; 256-wide tiles
// have no registers to hold them over a main loop and merge before it, in
// launches of one tile per workgroup.
bool linear_merges_stats(int64_t M, int N, int K, int parts, int n_cus) {
  if (parts > RING_MAX_PARTS) return false;
  const Choice c = linear_family(M, N, K, n_cus);
  switch (c.family) {
    case FAMILY_RING: return true;
    case FAMILY_MID: return (M + 127) / 128 * (N / 128) <= 8 * (int64_t)n_cus;
    case FAMILY_WIDE: return (M + c.rows - 1) / c.rows * (N / 256) <= n_cus;
    default: return false;
  }
}

hipError_t launch_linear(const uint16_t* X, const uint16_t* W, const float* bias, const uint16_t* R,
                         uint16_t* Y, int64_t M, int N, int K, int epi, const LinearExtra& ex,
                         hipStream_t stream) {
  if (M <= 0) return hipSuccess;
  const bool factors = epi == EPI_FOLD || epi == EPI_FOLD_GELU || epi == EPI_LNRES_STATS;
  if (factors && !ex.rows_in && !linear_merges_stats(M, N, K, ex.parts_in, ex.n_cus))
    return hipErrorInvalidValue;
  const auto [family, rows] = linear_family(M, N, K, ex.n_cus);
  if (family == FAMILY_RING)
    return launch_linear_ring(ring_tile(M, N, ex.n_cus), X, W, bias, R, Y, M, N, K, epi, ex, stream);
  if (family == FAMILY_MID) return launch_mid(X, W, bias, R, Y, M, N, N, K, epi, ex, stream);
  hipError_t e = launch_linear_wide(rows, X, W, bias, R, Y, M, N, K, epi, ex, stream);
  if (e != hipSuccess || family == FAMILY_WIDE) return e;
  const int cols = N & ~255;
  LinearExtra rest = ex;
  if (ex.stats_out) rest.stats_out = ex.stats_out + (int64_t)(cols / STATS_WIDTH) * M;
  if (ex.col_s) rest.col_s = ex.col_s + cols;
  if (ex.gamma) rest.gamma = ex.gamma + cols;
  if (ex.beta) rest.beta = ex.beta + cols;
  return launch_mid(X, W + (int64_t)cols * K, bias + cols, R ? R + cols : nullptr, Y + cols, M, N,
                    N - cols, K, epi, rest, stream);
}

}  // namespace surge
