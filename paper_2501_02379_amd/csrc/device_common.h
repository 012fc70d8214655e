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

// Selection key |g|^2 = fl(fl(re*re) + fl(im*im)) in float32, one rounding per operation (the
// _rn intrinsics are never contracted into a fused multiply-add).  Non-negative floats order
// like their bit patterns, so the key is compared as an unsigned integer.
__device__ __forceinline__ uint32_t select_key(float2 e) {
  return __float_as_uint(__fadd_rn(__fmul_rn(e.x, e.x), __fmul_rn(e.y, e.y)));
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
