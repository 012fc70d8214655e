// Device helpers shared by the first and last kernels of a step (contract_mfma.hip, ends.hip): range-checked
// streaming of G and W tiles, the storage policies of the weights, AdamUpdate on a sparse entry.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "device_common.h"

namespace tgrad {

// q = n / d, exact for n * d < 2^32 (callers keep n < 2^17, d < 2^10).
// magic = ceil(2^32 / d); d == 1 is encoded as magic == 0.
__device__ __forceinline__ uint32_t div_magic(uint32_t n, uint32_t magic) {
  return magic ? __umulhi(n, magic) : n;
}

// Orders the LDS accesses of one wavefront across its lanes (LDS executes a wavefront's
// instructions in order; this only keeps the compiler from moving them across the point).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Zero in a vector register that the compiler can neither fold nor prove uniform: an index built
// with it is loaded per lane (vector memory), not through the scalar cache.
__device__ __forceinline__ int opaque_zero() {
  int z = 0;
  asm volatile("" : "+v"(z));
  return z;
}

// Coefficients of the (re, im) parts of input element k for real output column (m, p):
// re(F x) = fr xr - fi xi,  im(F x) = fi xr + fr xi.
__device__ __forceinline__ float2 column_coef(float2 f, int p) {
  return p ? make_float2(f.y, f.x) : make_float2(f.x, -f.y);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_buffer(const void* base, uint32_t bytes) {
  // untyped buffer, stride 0: an access at offset >= bytes returns zero (loads) or is dropped (stores)
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}
// Two consecutive gradient elements as a buffer load returns them (one register tuple), and their
// float32 image in LDS.
template <int DT> struct BufPair;
template <> struct BufPair<TGRAD_C64> {
  typedef u32x4 type;
  static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, int voff) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 2);   // cache policy: non-temporal
  }
  static __device__ __forceinline__ void commit(float* dst, const type& v) { *reinterpret_cast<type*>(dst) = v; }
};
template <> struct BufPair<TGRAD_CBF16> {
  typedef u32x2 type;
  static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, int voff) {
    return __builtin_amdgcn_raw_buffer_load_b64(r, voff, 0, 2);    // cache policy: non-temporal
  }
  static __device__ __forceinline__ void commit(float* dst, const type& v) {   // a bf16 is the upper half of a float32
    u32x4 w;
    w.x = v.x << 16;
    w.y = v.x & 0xFFFF0000u;
    w.z = v.y << 16;
    w.w = v.y & 0xFFFF0000u;
    *reinterpret_cast<u32x4*>(dst) = w;
  }
};

struct SparseAdam {
  const int32_t* omega;
  const uint32_t* tile_start;
  const float2* gs;
  float2* ms;
  float* vs;
  float beta1, beta2;
  float scale, eps;     // N_S scaled by -lr lambda is scale m / (sqrt(v) + eps), both bias corrections folded in (sparse_adam)
  int k_last;           // max(k, 1) - 1: a support position that is always safe to read
};

// m c1 / (sqrt(v c2) + eps) = (c1 / sqrt(c2)) m / (sqrt(v) + eps / sqrt(c2)): two multiplications and their
// roundings less per entry; the constants are formed in float64.
inline SparseAdam sparse_adam(const int32_t* omega, const uint32_t* tile_start, const float2* gs, float2* ms, float* vs,
                              float beta1, float beta2, double inv_c1, double inv_c2, float eps, float c_lambda,
                              int k_last) {
  const double root = sqrt(inv_c2);
  return SparseAdam{omega, tile_start, gs, ms, vs, beta1, beta2, (float)((double)c_lambda * inv_c1 / root),
                    (float)((double)eps / root), k_last};
}

// AdamUpdate on sparse entry j (value x at support position oj, moments mm / v_old) and
// tile[oj] += (-lr lambda) N_S[j]; `sD` is the flat LDS image of the W tile that starts at w_base.
__device__ __forceinline__ void sparse_adam_entry(const SparseAdam& sp, uint32_t j, int32_t oj, float2 x,
                                                  float2 mm, float v_old, int64_t w_base, float* sD) {
  mm.x = sp.beta1 * mm.x + (1.f - sp.beta1) * x.x;
  mm.y = sp.beta1 * mm.y + (1.f - sp.beta1) * x.y;
  const float vv = sp.beta2 * v_old + (1.f - sp.beta2) * (x.x * x.x + x.y * x.y);
  sp.ms[j] = mm;
  sp.vs[j] = vv;
  const float d = sp.scale / (sqrtf(vv) + sp.eps);
  const int e = (int)((int64_t)oj - w_base);
  sD[2 * e] += d * mm.x;
  sD[2 * e + 1] += d * mm.y;
}

// How the weight tensor is stored (section "Mixed precision training": weights may be kept in half
// precision while the optimizer states stay in full precision).  A "piece" is 16 bytes of the W tile:
// 2 complex64 elements, or 4 elements stored as bf16 (re, im) pairs.  apply() returns
// decay * w + d for the piece, d read from the float32 image `sD` of the tile's update; bf16 weights
// are widened exactly, updated in float32 and rounded once (nearest even).
template <int WDT> struct WStore;
template <> struct WStore<TGRAD_C64> {
  typedef float4 raw;
  static constexpr int kElems = 2;
  static __device__ __forceinline__ raw* tile(void* w, int64_t w_base) {
    return reinterpret_cast<raw*>(reinterpret_cast<float*>(w) + 2 * w_base);
  }
  static __device__ __forceinline__ raw apply(const raw o, const float* sD, int q, float decay) {
    const float4 d = reinterpret_cast<const float4*>(sD)[q];
    return make_float4(decay * o.x + d.x, decay * o.y + d.y, decay * o.z + d.z, decay * o.w + d.w);
  }
  static __device__ __forceinline__ void apply_one(void* w, int64_t e, const float* d, float decay) {
    float2* p = reinterpret_cast<float2*>(w) + e;
    const float2 o = *p;
    *p = make_float2(decay * o.x + d[0], decay * o.y + d[1]);
  }
};
template <> struct WStore<TGRAD_CBF16> {
  typedef uint4 raw;
  static constexpr int kElems = 4;
  static __device__ __forceinline__ raw* tile(void* w, int64_t w_base) {
    return reinterpret_cast<raw*>(reinterpret_cast<uint32_t*>(w) + w_base);
  }
  static __device__ __forceinline__ uint32_t one(uint32_t o, float dre, float dim, float decay) {
    return bf16_pack(decay * __uint_as_float(o << 16) + dre, decay * __uint_as_float(o & 0xFFFF0000u) + dim);
  }
  static __device__ __forceinline__ raw apply(const raw o, const float* sD, int q, float decay) {
    const float4 d0 = reinterpret_cast<const float4*>(sD)[2 * q];
    const float4 d1 = reinterpret_cast<const float4*>(sD)[2 * q + 1];
    return make_uint4(one(o.x, d0.x, d0.y, decay), one(o.y, d0.z, d0.w, decay), one(o.z, d1.x, d1.y, decay),
                      one(o.w, d1.z, d1.w, decay));
  }
  static __device__ __forceinline__ void apply_one(void* w, int64_t e, const float* d, float decay) {
    uint32_t* p = reinterpret_cast<uint32_t*>(w) + e;
    *p = one(*p, d[0], d[1], decay);
  }
};
__device__ __forceinline__ void claim_raw(float4& r) {
  asm volatile("" : "+v"(r.x), "+v"(r.y), "+v"(r.z), "+v"(r.w));
}
__device__ __forceinline__ void claim_raw(uint2& r) { asm volatile("" : "+v"(r.x), "+v"(r.y)); }
__device__ __forceinline__ void claim_raw(uint4& r) { asm volatile("" : "+v"(r.x), "+v"(r.y), "+v"(r.z), "+v"(r.w)); }
// 16-byte pieces of W through a buffer descriptor (range-checked by the hardware: no clamps, no lane
// masks), non-temporal
__device__ __forceinline__ void buffer_piece_load(float4& d, __amdgpu_buffer_rsrc_t r, int voff) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 2);
  d = make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
__device__ __forceinline__ void buffer_piece_load(uint4& d, __amdgpu_buffer_rsrc_t r, int voff) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 2);
  d = make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void buffer_piece_store(const float4& d, __amdgpu_buffer_rsrc_t r, int voff) {
  u32x4 v;
  v.x = __float_as_uint(d.x);
  v.y = __float_as_uint(d.y);
  v.z = __float_as_uint(d.z);
  v.w = __float_as_uint(d.w);
  __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, 0, 2);
}
__device__ __forceinline__ void buffer_piece_store(const uint4& d, __amdgpu_buffer_rsrc_t r, int voff) {
  u32x4 v;
  v.x = d.x;
  v.y = d.y;
  v.z = d.z;
  v.w = d.w;
  __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, 0, 2);
}

inline uint32_t magic_for(int d) {
  return d <= 1 ? 0u : (uint32_t)((0x100000000ull + (uint64_t)d - 1) / (uint64_t)d);
}

}  // namespace tgrad
