// Device-side types and helpers for the gfx950 kernels.
//
// Activations and weights are stored as bf16 bit patterns (uint16_t) in HBM;
// all arithmetic is fp32 (MFMA accumulates in fp32).  Conversions to bf16
// use the hardware's round-to-nearest-even (v_cvt_pk_bf16_f32).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace surge {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
// Native 16-byte vector (HIP's uint4 is a union-based struct, which keeps
// LLVM from turning register arrays of it into registers).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(((uint32_t)b) << 16);
}

// Two floats -> packed bf16 pair (low half = a).
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  bf16x2 v;
  v[0] = (__bf16)a;
  v[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, v);
}

// Eight bf16 in a uint4 -> eight floats.
__device__ __forceinline__ void unpack8(const uint4& u, float* f) {
  f[0] = __uint_as_float(u.x << 16);
  f[1] = __uint_as_float(u.x & 0xffff0000u);
  f[2] = __uint_as_float(u.y << 16);
  f[3] = __uint_as_float(u.y & 0xffff0000u);
  f[4] = __uint_as_float(u.z << 16);
  f[5] = __uint_as_float(u.z & 0xffff0000u);
  f[6] = __uint_as_float(u.w << 16);
  f[7] = __uint_as_float(u.w & 0xffff0000u);
}

__device__ __forceinline__ uint4 pack8(const float* f) {
  uint4 u;
  u.x = pack_bf16x2(f[0], f[1]);
  u.y = pack_bf16x2(f[2], f[3]);
  u.z = pack_bf16x2(f[4], f[5]);
  u.w = pack_bf16x2(f[6], f[7]);
  return u;
}

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& u) { return __builtin_bit_cast(bf16x8, u); }

// LDS rows of CPR 16-byte chunks (CPR = 8: 64 bf16, CPR = 4: 32 bf16); the
// logical chunk c of row r is stored at position c ^ f(r), with
//   CPR = 8: f(r) = (r & 7) ^ ((r >> 3) & 1),
//   CPR = 4: f(r) = ((r >> 1) & 3) ^ ((r >> 3) & 1).
// For reads of one logical chunk from 32 consecutive rows (lane l reads row
// l % 32).  The LDS serves a 16-byte read 16 lanes at a time over 64 banks,
// of each half wave lanes 0-3, 12-15 and 20-27 together, then the others; in
// either set every lane falls on a slot of its own in a 256-byte window.
// Returns the slot index (16-byte units).
template <int CPR>
__device__ __forceinline__ int swz(int row, int chunk) {
  static_assert(CPR == 8 || CPR == 4, "LDS rows of 64 or 32 bf16");
  if (CPR == 8) return row * 8 + (chunk ^ (row & 7) ^ ((row >> 3) & 1));
  return row * 4 + (chunk ^ ((row >> 1) & 3) ^ ((row >> 3) & 1));
}

// A wave copy instruction (below) fills 64 consecutive slots: lane l's slot
// is row l / CPR (+ 64/CPR per further copy), stored position l % CPR.  The
// logical chunk that belongs there, the same for every further copy when
// the copies of a wave start at rows that are multiples of 16:
//   CPR = 8: (l & 7) ^ (l >> 3) ^ (copy & 1)    (rows 8 apart per copy),
//   CPR = 4: (l & 3) ^ ((l >> 3) & 3) ^ (l >> 5).
template <int CPR>
__device__ __forceinline__ int copy_chunk(int lane, int copy) {
  if (CPR == 8) return (lane & 7) ^ (lane >> 3) ^ (copy & 1);
  return (lane & 3) ^ ((lane >> 3) & 3) ^ (lane >> 5);
}

// The same for reads of 16 rows x 4 chunks (the operands of 16x16x32 MFMAs:
// lane l reads chunk l / 16 of row l % 16), with f(r) = r & 7 (under the f
// above every bank of such a read would be asked for twice: 41 to 47 % of the
// LDS's busy cycles were conflicts, none are now).
__device__ __forceinline__ int swz16(int row, int chunk) {
  return row * 8 + (chunk ^ (row & 7));
}
__device__ __forceinline__ int copy_chunk16(int lane) { return (lane & 7) ^ (lane >> 3); }

// Direct global -> LDS copy of 16 bytes per lane (gfx950 global_load_lds):
// the wave's 64 lanes land contiguously at LDS byte address `lds` (wave
// uniform, passed in M0).  Inline assembly, so the waits are placed by the
// kernel itself; the compiler does not track these loads.
__device__ __forceinline__ void copy_to_lds16(const void* g, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, off"
      :
      : "v"(g), "s"(lds)
      : "memory", "m0");
}

// The same with 4 bytes per lane (256 bytes per wave instruction).
__device__ __forceinline__ void copy_to_lds4(const void* g, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dword %0, off"
      :
      : "v"(g), "s"(__builtin_amdgcn_readfirstlane(lds))
      : "memory", "m0");
}

__device__ __forceinline__ void copy_to_lds4_at(const void* sbase, uint32_t voff, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dword %0, %1"
      :
      : "v"(voff), "s"(sbase), "s"(__builtin_amdgcn_readfirstlane(lds))
      : "memory", "m0");
}

// The same copy from sbase + voff: sbase wave-uniform (scalar registers),
// voff a 32-bit byte offset per lane.
__device__ __forceinline__ void copy_to_lds16_at(const void* sbase, uint32_t voff, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1"
      :
      : "v"(voff), "s"(sbase), "s"(lds)
      : "memory", "m0");
}

// The same with every lane on or off by `mask` (wave-uniform, ~0 or 0), for
// copies that may have to be skipped without a branch between the MFMAs
// around them.  Needs all 64 lanes active.  lane_mask makes such a mask and
// keeps it in a scalar register (the compiler folds a plain readfirstlane of
// a select away and may leave the select in a vector register).
__device__ __forceinline__ uint32_t lane_mask(bool on) {
  uint32_t v = on ? ~0u : 0u;
  asm volatile("" : "+v"(v));
  return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ void copy_to_lds16_if(const void* sbase, uint32_t voff, uint32_t lds,
                                                 uint32_t mask) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_mov_b32 exec_lo, %3\n\t"
      "s_mov_b32 exec_hi, %3\n\t"
      "global_load_lds_dwordx4 %0, %1\n\t"
      "s_mov_b64 exec, -1"
      :
      : "v"(voff), "s"(sbase), "s"(lds), "s"(mask)
      : "memory", "m0");
}

// The same copy from a wave-uniform base: lane l fetches the 16 bytes at
// base + 16 l (a 32-bit lane offset added to a scalar base, computed inside
// the statement so that no per-lane address has to stay live around it).
// `lds` must be wave-uniform.
__device__ __forceinline__ void copy_lanes_to_lds16(const void* base, uint32_t lds) {
  uint32_t voff;
  asm volatile(
      "v_mbcnt_lo_u32_b32 %0, -1, 0\n\t"
      "v_mbcnt_hi_u32_b32 %0, -1, %0\n\t"
      "v_lshlrev_b32 %0, 4, %0\n\t"
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1"
      : "=&v"(voff)
      : "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds))
      : "memory", "m0");
}

__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// A row's LayerNorm factors (rstd, -mean rstd) from its `parts` equal-width
// statistics partials (mean, biased variance), part(p): the row's mean is
// the average of the partial means, its variance the average partial
// variance plus the variance of the partial means.
//
// With MAXP > 0 (parts <= MAXP) every partial is loaded before any is used,
// so the loads' latencies overlap; MAXP = 0 takes any count.  Both forms sum
// in the same order.
template <int MAXP, class Part>
__device__ __forceinline__ float2 ln_row_factors(Part part, int parts, float eps) {
  float sm = 0.0f, sv = 0.0f, sd = 0.0f;
  const float inv_p = 1.0f / (float)parts;
  float mu;
  if constexpr (MAXP > 0) {
    float2 v[MAXP];
#pragma unroll
    for (int p = 0; p < MAXP; ++p)
      if (p < parts) v[p] = part(p);
#pragma unroll
    for (int p = 0; p < MAXP; ++p)
      if (p < parts) {
        sm += v[p].x;
        sv += v[p].y;
      }
    mu = sm * inv_p;
#pragma unroll
    for (int p = 0; p < MAXP; ++p)
      if (p < parts) {
        const float dm = v[p].x - mu;
        sd = fmaf(dm, dm, sd);
      }
  } else {
    for (int p = 0; p < parts; ++p) {
      const float2 v = part(p);
      sm += v.x;
      sv += v.y;
    }
    mu = sm * inv_p;
    for (int p = 0; p < parts; ++p) {
      const float dm = part(p).x - mu;
      sd = fmaf(dm, dm, sd);
    }
  }
  const float rstd = 1.0f / sqrtf(fmaf(sv + sd, inv_p, eps));
  return make_float2(rstd, -mu * rstd);
}

// GELU, z Phi(z) = max(z, 0) - |z| Phi(-|z|), both signs of z alike.  The
// normal tail is taken as Phi(-x) = 2^P(x) with P of degree 7, the minimax
// fit of log2 Phi(-x) on [0, 6] in the weight x Phi(-x) that its error has in
// GELU (6.1e-8), with P(x) < -27.99 - (x - 6) / 2 beyond, so that large |z|
// give 0.  In fp32 the error of GELU is at most 3e-7 (4.5e-8 rms on normal z).
// Seven FMAs and one exponential, 13 instruction slots with the sign handling
// against 16 of the rational form of Abramowitz & Stegun 7.1.28 that it
// replaces (7.1e-7, 1.5e-7 rms), in GEMM epilogues that the VALU bounds.
__device__ __forceinline__ float gelu_erf(float z) {
  const float az = fabsf(z);
  float p = fmaf(-6.83212739e-7f, az, 4.04779173e-5f);
  p = fmaf(p, az, -8.00353608e-4f);
  p = fmaf(p, az, 8.14606494e-3f);
  p = fmaf(p, az, -5.34843244e-2f);
  p = fmaf(p, az, -4.58730205e-1f);
  p = fmaf(p, az, -1.15121208f);
  p = fmaf(p, az, -9.99992214e-1f);
  return fmaf(-az, __builtin_amdgcn_exp2f(p), fmaxf(z, 0.0f));
}

}  // namespace surge
