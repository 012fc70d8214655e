// Device helpers shared by the kernel files: element loads for the two gradient
// storage types and the float32 selection key.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tgrad_internal.h"

namespace tgrad {

constexpr int kWave = 64;

// One complex element as (re, im) float32.  DT = TGRAD_C64: interleaved float32 pairs.
// DT = TGRAD_CBF16: interleaved bfloat16 pairs; a bf16 is the upper half of a float32, so
// widening is exact (re sits in the low 16 bits of the little-endian 32-bit word).
template <int DT>
__device__ __forceinline__ float2 load_elem(const void* g, int64_t i) {
  if constexpr (DT == TGRAD_C64) {
    return reinterpret_cast<const float2*>(g)[i];
  } else {
    uint32_t raw = reinterpret_cast<const uint32_t*>(g)[i];
    return make_float2(__uint_as_float(raw << 16), __uint_as_float(raw & 0xFFFF0000u));
  }
}

// Elements 2p and 2p+1 with one vector load (the pair is 16-byte / 8-byte aligned because
// the tensor base is).  The caller guarantees 2p + 1 < I.
template <int DT>
__device__ __forceinline__ void load_pair(const void* g, int64_t p, float2& e0, float2& e1) {
  if constexpr (DT == TGRAD_C64) {
    float4 v = reinterpret_cast<const float4*>(g)[p];
    e0 = make_float2(v.x, v.y);
    e1 = make_float2(v.z, v.w);
  } else {
    uint2 v = reinterpret_cast<const uint2*>(g)[p];
    e0 = make_float2(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u));
    e1 = make_float2(__uint_as_float(v.y << 16), __uint_as_float(v.y & 0xFFFF0000u));
  }
}

// Selection key |g|^2 = fl(fl(re*re) + fl(im*im)) in float32, one rounding per operation: contraction into a fused multiply-add
// is switched off here (it is the compiler's default, also for __fmul_rn and __fadd_rn, which are plain operators; a key with the
// first square unrounded differs in the last bit for a sixth of all numbers, and ties and the last entries taken went by that).
// Non-negative floats order like their bit patterns, so the key is compared as an unsigned integer.
__device__ __forceinline__ uint32_t select_key(float2 e) {
#pragma clang fp contract(off)
  const float rr = e.x * e.x, ii = e.y * e.y;
  return __float_as_uint(rr + ii);
}

// Entries of a factor (row-major complex), zero where `in` is false: through a range-checked buffer, so that nothing
// about the load is conditional.  (Written as a select, U[in ? i : 0] becomes a branch around the load and a wait right
// behind it: a table of 32 entries per thread was 32 memory round trips.  k_mid with 128 x 64 factors 58 us, now 52; whole
// steps 16x16x8x5 17.0 -> 15.7, 90x77x45x23 70.8 -> 66.4, 128x128x64x33 201 -> 192, in bf16 142 -> 132.)
// The buffer starts at U and covers `entries` of it, at most 2 GB.
typedef __amdgpu_buffer_rsrc_t FactorRef;
__device__ __forceinline__ FactorRef factor_ref(const float2* U, int64_t entries) {
  const int64_t bytes = entries * 8 < 0x7FFFFFF8 ? entries * 8 : 0x7FFFFFF8;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(U), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float2 factor_entry(const FactorRef& f, int row, int col, int cols, bool in) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  const uint32_t off = in ? ((uint32_t)row * (uint32_t)cols + (uint32_t)col) * 8u : 0xFFFFFFF0u;
  const u2 v = __builtin_amdgcn_raw_buffer_load_b64(f, off, 0, 0);
  return make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
}

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4f mfma16(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ---- float32 products on the bf16 matrix instructions -------------------------------------------
// x = h + m + l with h the upper 8 bits of x, m = bf16(x - h), l = bf16(x - h - m): three times 8 bits hold all 24 of a
// float32, and a x b = hh + hm + mh + hl + lh + mm leaves out products below 2^-23 of it (ml, lm, ll: typically 2^-26).  Six
// v_mfma_f32_16x16x32_bf16 do the work of eight v_mfma_f32_16x16x4f32 in 96 cycles instead of 256, and, unlike those, beside
// vector instructions of another wavefront.  They add 32 products per rounding instead of 4, so sums come out closer to 64
// bits than before: relative error of a sum of K products of normal numbers, float32 instructions / these: K = 32 1.0e-7 /
// 4.4e-8, 128 2.1e-7 / 1.6e-7 (6.9e-8 with the five small terms summed apart), 1024 5.7e-7 / 4.8e-7.
// What float32 instructions did and these do not: numbers below 2^-110 lose their last bits (parts below 2^-133, the smallest
// bf16, are lost: an error of 8e-7 at 2^-114, 2e-4 at 2^-122; their squares are zero in float32, so AdamUpdate divides such a
// gradient by eps alone and the weights do not show it); an infinity becomes NaN, in both parts of its complex number (inf - inf; two complex products
// with finite factors made NaN of it before as well, and every step has more).
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32v4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32v2 __attribute__((ext_vector_type(2)));

// Two float32 -> bf16 pairs (first in the low half), rounded to nearest, ties to even, NaN to a quiet NaN: one
// v_cvt_pk_bf16_f32.  (In integer arithmetic it was 14 vector instructions per pair, and with bf16 weights those
// bounded the update: k_tail at 128x128x64x33 81 us, now 66.)
__device__ __forceinline__ uint32_t bf16_pack(float re, float im) {
  f32x2 v;
  v.x = re;
  v.y = im;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Eight real numbers of a lane as an operand: four dwords of two neighbouring numbers, for each of the three parts.
struct Split8 {
  u32v4 h, m, l;
};
// One dword of each part from a pair of numbers.  x - h is exact, and one v_dot2c_f32_bf16 per number: dot2(h, (-1, 0), x).
// (The constants are kept in registers: as an inline constant of the instruction, (-1, 0) would be read as a float32.)
// h is cut off, not rounded: to nearest, a number above 3.39e38 would be an infinity and the rest NaN, and limiting every
// number first cost 2 to 3 % of a step (128x128x128x65 743 us, 763).
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  uint32_t lo = 0x0000BF80u, hi = 0xBF800000u;
  asm("" : "+s"(lo), "+s"(hi));
  const bf16x2 n0 = __builtin_bit_cast(bf16x2, lo), n1 = __builtin_bit_cast(bf16x2, hi);
  h = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);   // the upper halves
  const bf16x2 hv = __builtin_bit_cast(bf16x2, h);
  a = __builtin_amdgcn_fdot2_f32_bf16(hv, n0, a, false);
  b = __builtin_amdgcn_fdot2_f32_bf16(hv, n1, b, false);
  m = bf16_pack(a, b);
  const bf16x2 mv = __builtin_bit_cast(bf16x2, m);
  a = __builtin_amdgcn_fdot2_f32_bf16(mv, n0, a, false);
  b = __builtin_amdgcn_fdot2_f32_bf16(mv, n1, b, false);
  l = bf16_pack(a, b);
}
__device__ __forceinline__ void split_at(Split8& s, int d, float2 v) {   // numbers 2 d, 2 d + 1
  uint32_t h, m, l;
  split_pair(v.x, v.y, h, m, l);
  s.h[d] = h;
  s.m[d] = m;
  s.l[d] = l;
}
// (re, im) pairs -> (im, re), and -> (re, -im): the second operands of a complex product
__device__ __forceinline__ u32v4 swap_pairs(u32v4 v) {
#pragma unroll
  for (int d = 0; d < 4; ++d) v[d] = __builtin_amdgcn_alignbit(v[d], v[d], 16);
  return v;
}
__device__ __forceinline__ u32v4 conj_pairs(u32v4 v) { return v ^ 0x80000000u; }
__device__ __forceinline__ Split8 swap_pairs(const Split8& s) { return Split8{swap_pairs(s.h), swap_pairs(s.m), swap_pairs(s.l)}; }
__device__ __forceinline__ Split8 conj_pairs(const Split8& s) { return Split8{conj_pairs(s.h), conj_pairs(s.m), conj_pairs(s.l)}; }

// D[i = 4 g + r][j = c] += sum over the 32 slots (g, s): A[c][(g, s)] B[(g, s)][c]; which index of the sum a slot stands
// for is the caller's choice, the same for both operands.
__device__ __forceinline__ v4f mfma_bf(u32v4 a, u32v4 b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// N independent products with the same A: the six terms, smallest first
template <int N>
__device__ __forceinline__ void mfma_split(v4f* acc, const Split8& a, const Split8* b) {
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a.l, b[i].h, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a.h, b[i].l, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a.m, b[i].m, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a.m, b[i].h, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a.h, b[i].m, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a.h, b[i].h, acc[i]);
}

// ... with the same B
template <int N>
__device__ __forceinline__ void mfma_split_b(v4f* acc, const Split8* a, const Split8& b) {
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a[i].l, b.h, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a[i].h, b.l, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a[i].m, b.m, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a[i].m, b.h, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a[i].h, b.m, acc[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = mfma_bf(a[i].h, b.h, acc[i]);
}
// One product over 16 slots (dwords 0 and 1 of the operands)
__device__ __forceinline__ v4f mfma_bf_half(u32v4 a, u32v4 b, v4f c) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  const u32v2 al = {a.x, a.y}, bl = {b.x, b.y};
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, al), __builtin_bit_cast(s16x4, bl), c, 0, 0, 0);
}
__device__ __forceinline__ void mfma_split_half(v4f& acc, const Split8& a, const Split8& b) {
  acc = mfma_bf_half(a.l, b.h, acc);
  acc = mfma_bf_half(a.h, b.l, acc);
  acc = mfma_bf_half(a.m, b.m, acc);
  acc = mfma_bf_half(a.m, b.h, acc);
  acc = mfma_bf_half(a.h, b.m, acc);
  acc = mfma_bf_half(a.h, b.h, acc);
}

// dst[0 .. n) = gen(e) by a workgroup, 8 loads per thread in flight
template <typename Gen>
__device__ __forceinline__ void stage_table(float2* dst, int n, int tid, int nthreads, Gen gen) {
  for (int e0 = tid; e0 < n; e0 += nthreads * 8) {
    float2 f[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) f[u] = gen(e0 + u * nthreads < n ? e0 + u * nthreads : e0);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (e0 + u * nthreads < n) dst[e0 + u * nthreads] = f[u];
  }
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Number of set bits of `b` strictly below this lane.
__device__ __forceinline__ int popc_below(uint64_t b, int lane) {
  return __popcll(b & ((1ull << lane) - 1ull));
}

}  // namespace tgrad
