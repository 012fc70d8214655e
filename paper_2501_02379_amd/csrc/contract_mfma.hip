// Mode-n products of the per-step path of Algorithm 1 on the fp32 matrix cores
// (v_mfma_f32_32x32x2f32), for low-rank compression  g_L = (G - Sparse(G, Omega)) x_n U^(n)H
// and reconstruction  G~_L = N_L x_n U^(n)  (section "Low-rank gradient tensor decomposition",
// appendix "Tensor Operations and Notation", mode-k product).
//
// A complex contraction is run as a real one without padding or wasted flops: a tensor of
// interleaved (re, im) float32 pairs is used as it lies in memory, and the factor is expanded to
// its 2 x 2 real blocks.  With F = Fr + i Fi and X = Xr + i Xi,
//   re(F X) = Fr Xr - Fi Xi,   im(F X) = Fr Xi + Fi Xr,
// i.e. 4 real multiply-adds per complex multiply-add on either layout below.
//
// The kernels:
//  (the modes between: mid.hip, core2.hip; both ends on 16 x 16 tiles: ends.hip; the last mode alone, up to 72 entries: rows.hip)
//  k_lproj    contracts the LAST mode of the gradient itself (first compression stage): a
//             flat tile of rows is staged in LDS, the entries of the support Omega that fall
//             in the tile are handed to the sparse branch (gather) and zeroed (this is
//             G - Sparse(G, Omega) without a second pass over G), then 32 rows per wavefront
//             go through the matrix cores.  With FUSE it also contracts mode N-1 (the tile's mode-N
//             result, still in the accumulators, is the operand of the next contraction);
//             k_lproj_flat is that fused form for odd last extents.
//  k_lupdate  the last reconstruction stage fused with everything that touches W: expands the
//             last mode into an LDS tile, runs AdamUpdate on the sparse values of the tile
//             and adds lambda N_S into it, then streams W <- W (1 - lr wd) - lr tile with
//             16-byte accesses.  k_lupdate_fused also expands mode N-1 in front of it.
//  k_mfma_probe_*  register-resident matrix-core loops (calibration of the reported fractions).
//
// Operand layout of v_mfma_f32_32x32x2f32 (D = A B + C, A 32 x 2, B 2 x 32, 64 lanes):
//   lane l supplies A[l % 32][l / 32] and B[l / 32][l % 32];
//   register r of lane l receives D[(r % 4) + 8 (r / 4) + 4 (l / 32)][l % 32].
#include <type_traits>

#include "device_common.h"
#include "end_common.h"
#include "launch_util.h"

namespace tgrad {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ v16f mfma32(float a, float b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int d_row(int r, int half) { return (r & 3) + 8 * (r >> 2) + 4 * half; }

// -------------------------------------------------------------------------------------------
// Register-resident matrix-core loops: what the matrix cores of this chip deliver when nothing else
// is in the way (no memory, no LDS, operands constant).  The reference point for the matrix-core
// fractions of the kernels below, next to the published peaks.  Four independent accumulators per
// wavefront, two wavefronts per SIMD.
typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kProbeChains = 4;
constexpr int kProbeUnroll = 64;             // rounds per trip of the loop (the loop's own bookkeeping is then negligible)
__global__ __launch_bounds__(256) void k_mfma_probe_f32(float* sink, int64_t iters, float a, float b) {
  v16f acc[kProbeChains];
#pragma unroll
  for (int c = 0; c < kProbeChains; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[c][r] = 0.f;
  for (int64_t i = 0; i < iters; i += kProbeUnroll) {          // (iters is a multiple of kProbeUnroll: host)
#pragma unroll
    for (int u = 0; u < kProbeUnroll; ++u)
#pragma unroll
      for (int c = 0; c < kProbeChains; ++c) acc[c] = mfma32(a, b, acc[c]);
  }
  float t = 0.f;
#pragma unroll
  for (int c = 0; c < kProbeChains; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) t += acc[c][r];
  if (t == 12345.678f) sink[0] = t;                            // (never: a b iters is not that number; keeps the loop alive)
}
__global__ __launch_bounds__(256) void k_mfma_probe_f64(float* sink, int64_t iters, double a, double b) {
  v4d acc[kProbeChains];
#pragma unroll
  for (int c = 0; c < kProbeChains; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[c][r] = 0.;
  for (int64_t i = 0; i < iters; i += kProbeUnroll) {
#pragma unroll
    for (int u = 0; u < kProbeUnroll; ++u)
#pragma unroll
      for (int c = 0; c < kProbeChains; ++c) acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[c], 0, 0, 0);
  }
  double t = 0.;
#pragma unroll
  for (int c = 0; c < kProbeChains; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) t += acc[c][r];
  if (t == 12345.678) sink[0] = (float)t;
}

// -------------------------------------------------------------------------------------------
// Shared by the two last-mode kernels.  The tensor seen as (A rows, L complex per row) is cut
// into flat tiles of 32 rows (one matrix-core tile); tile t holds elements [32 t L, 32 (t + 1) L).
// `tile_start[t]` = number of support entries below 32 t L (Omega is ascending), so tile t owns
// Omega[tile_start[t] .. tile_start[t + 1]).
//
// A tile belongs to ONE wavefront from its first load to its last store, and the LDS slice it
// is staged in is private to that wavefront.  The wavefronts of a workgroup therefore never
// meet at a barrier after the factor table is staged: each runs its own load / matrix-core /
// store pipeline and the hardware overlaps them.  Workgroups have 4 wavefronts because a
// workgroup's wavefronts are spread over the 4 SIMDs of a compute unit starting at the first
// one: smaller workgroups leave the matrix cores of the last SIMDs idle.
constexpr int kTileRows = 32;

// Factor table in LDS: sF[k * ld + m] = scale * F[m, k] as (fr, fi), ld = 16 NT, zero for k >= K
// or m >= M.  PROJECT: F[m, k] = conj(U[k, m]); otherwise F[m, k] = U[m, k].
template <bool PROJECT>
__device__ __forceinline__ void stage_factor_table(float2* sF, const float2* __restrict__ U, int rn, int K,
                                                   int M, int krows, int ld, int tid, int nthreads,
                                                   float scale = 1.f) {
  for (int e = tid; e < krows * ld; e += nthreads) {
    const int k = e / ld, m = e - k * ld;
    float2 f = make_float2(0.f, 0.f);
    if (k < K && m < M) {
      if (PROJECT) {
        const float2 u = U[(int64_t)k * rn + m];
        f = make_float2(u.x, -u.y);
      } else {
        f = U[(int64_t)m * rn + k];
      }
    }
    sF[e] = make_float2(scale * f.x, scale * f.y);
  }
}
// Two consecutive gradient elements as they lie in memory (complex64: 16 bytes, bf16 pairs: 8).
template <int DT> struct RawPair;
template <> struct RawPair<TGRAD_C64> { typedef float4 type; };
template <> struct RawPair<TGRAD_CBF16> { typedef uint2 type; };

// Streaming accesses.  G is read once per step and W is read and written once per step; marked
// non-temporal they neither push the small reused operands (factor tables, intermediate tensors) out
// of the caches nor leave a cache full of dirty lines behind for the next kernel to wait on.
typedef float f32x4nt __attribute__((ext_vector_type(4)));
typedef float f32x2nt __attribute__((ext_vector_type(2)));
template <typename R>
__device__ __forceinline__ R nt_load(const R* p) {
  if constexpr (sizeof(R) == 16)
    return __builtin_bit_cast(R, __builtin_nontemporal_load(reinterpret_cast<const f32x4nt*>(p)));
  else
    return __builtin_bit_cast(R, __builtin_nontemporal_load(reinterpret_cast<const f32x2nt*>(p)));
}
template <typename R>
__device__ __forceinline__ void nt_store(R* p, const R& v) {
  static_assert(sizeof(R) == 16, "16-byte pieces");
  __builtin_nontemporal_store(__builtin_bit_cast(f32x4nt, v), reinterpret_cast<f32x4nt*>(p));
}

template <int DT>
__device__ __forceinline__ typename RawPair<DT>::type load_raw_pair(const void* g, int64_t p) {
  return nt_load(reinterpret_cast<const typename RawPair<DT>::type*>(g) + p);
}
template <int DT>
__device__ __forceinline__ void decode_raw(const typename RawPair<DT>::type& raw, float2& e0, float2& e1) {
  if constexpr (DT == TGRAD_C64) {
    e0 = make_float2(raw.x, raw.y);
    e1 = make_float2(raw.z, raw.w);
  } else {                                   // a bf16 is the upper half of a float32: widening is exact
    e0 = make_float2(__uint_as_float(raw.x << 16), __uint_as_float(raw.x & 0xFFFF0000u));
    e1 = make_float2(__uint_as_float(raw.y << 16), __uint_as_float(raw.y & 0xFFFF0000u));
  }
}


constexpr int kTileBatch = 17;            // 2-element pieces per lane in flight while a tile is staged (the most;
                                          // narrower last modes use 9 or 5: a tile of K-wide rows has K / 4 per lane)
constexpr int kJUnroll = 4;               // row pairs whose LDS operands are fetched ahead of their MFMAs
constexpr int kCoefPairs = 33;            // fused first stage: most row pairs whose coefficients stay in registers
constexpr int kCoefPairsShort = 17;       // ... and the variant for short last modes (I_N <= 34)

// k_lproj: out[a, m] = sum_k conj(U[k, m]) (G - Sparse(G, Omega))[a, k];  gs[j] = G[Omega_j].
// Wavefront w of workgroup b walks tiles b W + w, + gridDim.x W, ...; the global loads of its next
// tile are issued before the matrix-core phase of the current one.
// Matrix-core step (j, part): lanes 0..31 feed element k = 2 j, lanes 32..63 element k = 2 j + 1
// of their row (part = re, then im).  The loops carry no guards (a guarded, branchy loop ran the
// matrix cores at less than half their rate): for odd K the last pair reads element k = K of the
// row, whose coefficients are zero and whose LDS slot always holds a finite value.
//
// FUSE: the next compression stage (mode N-1, extent 32 S, rank M2 <= 32) runs on the matrix-core
// result while it is still in registers.  A wavefront then walks whole slabs (the S consecutive
// tiles that share all leading indices): the 32 x 32 result tile of stage one is, as it lies in the
// accumulator registers, the B operand of  D2[m2, (m3, p)] += F2[m2, i2] Y[i2, (m3, p)]  (register r
// holds rows d_row(r, 0) / d_row(r, 1) of the tile in the two lane halves = one row pair); the
// re/im swap of Y for the imaginary part of F2 is a swap of neighbouring lanes (DPP).  D2 is
// stored once per slab; the intermediate tensor between the two stages never exists.
struct FusedNext {
  const float2* fpad;   // conj(U^(N-1)[i2, m2]) as (re, im), zero for m2 >= M2, in operand order (k_pack_fused_factor)
  float* out;           // (slabs, M2, M) complex, row-major
  int S;                // tiles per slab; 1 when nothing is fused
  int M2;
};

template <int DT, int W, int NTB, bool FLAT, bool FUSE, int CP, int TB>
__global__ __launch_bounds__(64 * W, 2) void k_lproj(const void* __restrict__ g,
                                                     const int32_t* __restrict__ omega,
                                                     const uint32_t* __restrict__ tile_start,
                                                     float2* __restrict__ gs, const float2* __restrict__ U,
                                                     int rn, int64_t A, int K, int M, uint32_t magicK,
                                                     int64_t ntiles, float* __restrict__ out,
                                                     FusedNext fz) {
  typedef typename RawPair<DT>::type Raw;
  constexpr int T = 64 * W;
  extern __shared__ float smem[];
  constexpr bool flat = FLAT;                                  // odd K: the LDS image is the memory image
  const int stride = 2 * K + (flat ? 0 : 2);                   // floats per LDS row; stride / 2 is odd
  const int slice = kTileRows * stride + 2;                    // floats per wavefront (even)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // in a scalar register: tile bookkeeping stays scalar
  float* sX = smem + wave * slice;
  float2* sF = reinterpret_cast<float2*>(smem + W * slice);
  const int J = (K + 1) >> 1;
  const int N2 = 2 * M;
  const int NT = (N2 + 31) >> 5;
  const int ld = 16 * NT;
  for (int e = lane; e < slice; e += 64) sX[e] = 0.f;          // pads and never-staged rows stay finite
  stage_factor_table<true>(sF, U, rn, K, M, 2 * J, ld, tid, T);
  __syncthreads();                                             // the only workgroup barrier
  // FUSE (one column tile, J <= CP): the lane's first-stage coefficients - one (re, im) pair per
  // row pair - do not depend on the tile, so they live in registers for the whole kernel and the
  // matrix-core loop reads only its A operand from LDS.  Row pairs past J carry zeros.
  float2 creg[FUSE ? CP : 1];
  if constexpr (FUSE) {
    const int c0 = lane & 31, h0 = lane >> 5;
    const float2* fl0 = sF + h0 * ld + (c0 >> 1);
#pragma unroll
    for (int j = 0; j < CP; ++j)
      creg[j] = j < J ? column_coef(fl0[2 * j * ld], c0 & 1) : make_float2(0.f, 0.f);
  }

  const int64_t I = A * K;
  const int tile_elems = kTileRows * K;
  // Tile sequence of this wavefront: slabs wg, wg + nw, ... and inside a slab its S tiles in order
  // (S = 1 without fusion, where a slab is a tile).
  const int S = FUSE ? fz.S : 1;
  const int64_t nslabs = (ntiles + S - 1) / S;
  const int64_t nw = (int64_t)gridDim.x * W;
  int64_t slab = (int64_t)blockIdx.x * W + wave;
  int ts = 0;
  if (slab >= nslabs) return;
  auto advance = [&](int64_t& sl, int& t) {                    // next position of the sequence
    if (t + 1 < S) { t += 1; } else { t = 0; sl += nw; }
  };

  Raw raw[TB];
  int32_t my_om = -1;
  // issue the first batch of tile `t` (its support range is [j0, j1)) into raw / my_om.  The loads
  // are unconditional (indices past the tile are clamped onto its last pair): a conditional load
  // would be followed by a wait and a register copy.
  auto issue = [&](int64_t t, uint32_t j0, uint32_t j1) {
    const int64_t e_base = t * tile_elems;
    const int n_e = (int)((I - e_base) < tile_elems ? (I - e_base) : tile_elems);
    const int npairs = n_e >> 1;                               // >= 1: the host keeps K >= 2 here
#pragma unroll
    for (int i = 0; i < TB; ++i) {
      const int pi = lane + i * 64;
      raw[i] = load_raw_pair<DT>(g, (e_base >> 1) + (pi < npairs ? pi : npairs - 1));
    }
    my_om = (j0 + lane < j1) ? omega[j0 + lane] : -1;
  };
  // element pair at flat offset e0 of the tile -> LDS
  auto commit_pair = [&](const Raw& rw, int e0) {
    float2 v0, v1;
    decode_raw<DT>(rw, v0, v1);
    if (flat) {
      *reinterpret_cast<float4*>(&sX[2 * e0]) = make_float4(v0.x, v0.y, v1.x, v1.y);
    } else {
      const uint32_t r0 = div_magic((uint32_t)e0, magicK);
      const uint32_t c0 = (uint32_t)e0 - r0 * (uint32_t)K;
      const bool wrap = c0 + 1 == (uint32_t)K;
      const uint32_t r1 = wrap ? r0 + 1 : r0;
      const uint32_t c1 = wrap ? 0u : c0 + 1;
      *reinterpret_cast<float2*>(&sX[r0 * stride + 2 * c0]) = v0;
      *reinterpret_cast<float2*>(&sX[r1 * stride + 2 * c1]) = v1;
    }
  };

  // The support ranges are fetched with per-lane (vector) loads on purpose: a scalar load shares
  // its wait counter with the LDS reads of the matrix-core phase and would stall its first step.
  const int vzero = opaque_zero();
  int64_t tile = slab * S;
  int64_t nslab = slab;
  int nts = ts;
  advance(nslab, nts);
  bool have_next = nslab < nslabs;
  int64_t nxt = have_next ? nslab * S + nts : tile;            // past the end: reload the current tile (unused)
  uint32_t cj0 = tile_start[tile + vzero], cj1 = tile_start[tile + 1 + vzero];
  uint32_t nj0 = tile_start[nxt + vzero], nj1 = tile_start[nxt + 1 + vzero];
  issue(tile, cj0, cj1);
  v16f acc2;                                                   // FUSE: second-stage accumulator of the slab
#pragma unroll
  for (int r = 0; r < 16; ++r) acc2[r] = 0.f;
  while (true) {
    const int64_t e_base = tile * tile_elems;
    const int n_e = (int)((I - e_base) < tile_elems ? (I - e_base) : tile_elems);
    wave_sync();                                               // previous tile's LDS reads are done
    // Opaque copy of the lane id: everything addressed through it is recomputed per tile (a few
    // VALU operations) instead of being hoisted into dozens of long-lived registers, which
    // would spill - and a spill reload waits for every load in flight.
    int lane_now = lane;
    asm volatile("" : "+v"(lane_now));
    const int col = lane_now & 31, half = lane_now >> 5;
    const float* xa = sX + col * stride + 2 * half;            // the lane's own row, its half of each pair
    const float2* fl = sF + half * ld + (col >> 1);
    const int part = col & 1;
    // one wait for the whole batch (the only memory operations issued after it were loads)
    asm volatile("" : "+v"(my_om));
#pragma unroll
    for (int i = 0; i < TB; ++i) claim_raw(raw[i]);
    const int npairs = n_e >> 1;
#pragma unroll
    for (int i = 0; i < TB; ++i) {
      const int pi = lane_now + i * 64;
      if (pi < npairs) commit_pair(raw[i], 2 * pi);
    }
    for (int pi = lane + TB * 64; pi < npairs; pi += 64)          // long rows: the rest, unpipelined
      commit_pair(load_raw_pair<DT>(g, (e_base >> 1) + pi), 2 * pi);
    if ((n_e & 1) && lane == 0) {                              // odd element count: the last one alone
      const int e = n_e - 1;
      const float2 v = load_elem<DT>(g, e_base + e);
      const uint32_t r = div_magic((uint32_t)e, magicK);
      *reinterpret_cast<float2*>(&sX[r * stride + 2 * ((uint32_t)e - r * (uint32_t)K)]) = v;
    }
    // ---- second-stage factor operands of this tile (FUSE): small, cache-resident; issued before
    //      the next tile's loads so that waiting for them leaves those in flight ----
    float2 f2s[FUSE ? 16 : 1];
    if constexpr (FUSE) {
      const float4* fp = reinterpret_cast<const float4*>(fz.fpad) + (size_t)ts * 8 * 64 + lane_now;
#pragma unroll
      for (int rp = 0; rp < 8; ++rp) {
        const float4 f = fp[rp * 64];
        f2s[2 * rp] = make_float2(f.x, f.y);
        f2s[2 * rp + 1] = make_float2(f.z, f.w);
      }
    }
    // ---- the staging registers are free: the next tile's loads go in flight right away (its
    //      support range was fetched one tile earlier).  All unconditional: see `issue`. ----
    const int32_t cur_om = my_om;
    int64_t nnslab = nslab;
    int nnts = nts;
    advance(nnslab, nnts);
    const bool have_nn = have_next && nnslab < nslabs;
    const int64_t nn = have_nn ? nnslab * S + nnts : nxt;
    issue(nxt, nj0, nj1);
    const uint32_t nnj0 = tile_start[nn + vzero], nnj1 = tile_start[nn + 1 + vzero];
    wave_sync();
    // ---- Sparse(G, Omega) of this tile: hand the values over, then remove them ----
    // (the first 64 entries of the tile were prefetched with it: the common path loads nothing, so
    // it never waits for the loads just issued; longer ranges take the rare second loop)
    auto take_entry = [&](uint32_t j, int32_t oj) {
      const uint32_t e = (uint32_t)((int64_t)oj - e_base);
      const uint32_t r = flat ? 0u : div_magic(e, magicK);
      float2* p = reinterpret_cast<float2*>(&sX[r * stride + 2 * (e - r * (uint32_t)K)]);
      gs[j] = *p;
      *p = make_float2(0.f, 0.f);
    };
    if (cj0 + lane < cj1) take_entry(cj0 + lane, cur_om);
    if (cj1 - cj0 > 64u)
      for (uint32_t j = cj0 + 64u + lane; j < cj1; j += 64) take_entry(j, omega[j]);
    wave_sync();
    // ---- the 32 rows through the matrix cores, NTB column tiles at a time ----
    const int64_t grow0 = tile * kTileRows;
    auto block = [&](int nt0, auto ntile_count) {
      constexpr int N = decltype(ntile_count)::value;
      v16f acc[N];
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
      const float2* fb = fl + 16 * nt0;
      int j = 0;
      if constexpr (FUSE) {
        // straight-line: CP row pairs, A operands fetched kJUnroll pairs ahead; pairs past J re-read
        // the last one and meet zero coefficients
        const int jlast = J - 1;
        float2 a2[kJUnroll];
#pragma unroll
        for (int u = 0; u < kJUnroll; ++u) a2[u] = *reinterpret_cast<const float2*>(xa + 4 * (u < jlast ? u : jlast));
#pragma unroll
        for (int jj = 0; jj < CP; ++jj) {
          const float2 a = a2[jj % kJUnroll];
          if (jj + kJUnroll < CP) {
            const int jn = jj + kJUnroll;
            a2[jj % kJUnroll] = *reinterpret_cast<const float2*>(xa + 4 * (jn < jlast ? jn : jlast));
          }
          acc[0] = mfma32(a.x, creg[jj].x, acc[0]);
          acc[0] = mfma32(a.y, creg[jj].y, acc[0]);
        }
        j = J;
      }
      for (; j + kJUnroll <= J; j += kJUnroll) {
        float2 a2[kJUnroll], f2[kJUnroll][N];
#pragma unroll
        for (int u = 0; u < kJUnroll; ++u) {
          a2[u] = *reinterpret_cast<const float2*>(xa + 4 * (j + u));
#pragma unroll
          for (int i = 0; i < N; ++i) f2[u][i] = fb[2 * (j + u) * ld + 16 * i];
        }
#pragma unroll
        for (int u = 0; u < kJUnroll; ++u)
#pragma unroll
          for (int i = 0; i < N; ++i) {
            const float2 b2 = column_coef(f2[u][i], part);
            acc[i] = mfma32(a2[u].x, b2.x, acc[i]);
            acc[i] = mfma32(a2[u].y, b2.y, acc[i]);
          }
      }
      for (; j < J; ++j) {
        const float2 a2 = *reinterpret_cast<const float2*>(xa + 4 * j);
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const float2 b2 = column_coef(fb[2 * j * ld + 16 * i], part);
          acc[i] = mfma32(a2.x, b2.x, acc[i]);
          acc[i] = mfma32(a2.y, b2.y, acc[i]);
        }
      }
      if constexpr (FUSE) {                                    // NT == 1, N == 1
        asm volatile("" : "+v"(f2s[0].x));                     // the factor operands are claimed here
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float y = acc[0][r];
          const float sw = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(y), 0xB1, 0xF, 0xF, true));
          const float yj = part ? sw : -sw;                    // (Y J): re column <- -im, im column <- re
          acc2 = mfma32(f2s[r].x, y, acc2);
          acc2 = mfma32(f2s[r].y, yj, acc2);
        }
        if (ts == S - 1) {                                     // slab complete: D2 -> out[slab, m2, c]
          float* o = fz.out + (size_t)slab * fz.M2 * N2 + col;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int m2 = d_row(r, half);
            if (m2 < fz.M2 && col < N2) o[m2 * N2] = acc2[r];
            acc2[r] = 0.f;
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const int c = 32 * (nt0 + i) + col;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int64_t grow = grow0 + d_row(r, half);
            if (grow < A && c < N2) out[grow * N2 + c] = acc[i][r];
          }
        }
      }
    };
    if constexpr (FUSE) {
      __builtin_amdgcn_s_setprio(1);                           // matrix-core phase: ahead of the other wavefront's loads and stores
      block(0, std::integral_constant<int, 1>());              // exactly one column tile (and no loop around the
    } else {                                                   // claim of f2s: a loop preheader would drain all loads)
      int nt0 = 0;
      for (; nt0 + NTB <= NT; nt0 += NTB) block(nt0, std::integral_constant<int, NTB>());
      if (NTB > 1)
        for (; nt0 < NT; ++nt0) block(nt0, std::integral_constant<int, 1>());
    }
    if constexpr (FUSE) __builtin_amdgcn_s_setprio(0);
    if (!have_next) break;
    tile = nxt;
    slab = nslab;
    ts = nts;
    nxt = nn;
    nslab = nnslab;
    nts = nnts;
    have_next = have_nn;
    cj0 = nj0;
    cj1 = nj1;
    nj0 = nnj0;
    nj1 = nnj1;
  }
}

// -------------------------------------------------------------------------------------------
// k_lproj_flat: k_lproj<.., FUSE> for odd last extents (the LDS image of a tile is its memory image),
// written so that everything a wavefront does OUTSIDE its matrix-core phase is scalar, LDS or
// vector-memory work with loop-invariant vector registers.  fp32 MFMA instructions run on the SIMD's
// vector ALU: while one wavefront of a SIMD is in its matrix-core phase, a vector-ALU instruction of
// the other one does not issue, so address arithmetic, clamps and lane masks in the staging phase
// serialise the two wavefronts instead of overlapping them.  Here
//  - the tile is fetched with buffer loads: the descriptor (scalar registers) carries the tile's
//    base and size, lanes past the tile's end read zero without touching memory, and the lane's
//    offset is one invariant register;
//  - every lane commits what it loaded (the slice has room for TB x 64 pieces; the host picks TB so
//    that they cover the tile: TB x 64 >= 16 K), so no lane masks;
//  - support ranges, factor operands and results go through scalar bases + invariant lane offsets.
// Same tile sequence and the same arithmetic, in the same order, as k_lproj<.., FUSE>.
// floats of LDS per wavefront: the tile (32 rows of K complex + one pad pair for the row pair past
// an odd K) or, if larger, what TB x 64 committed pieces cover; a multiple of 4 (16-byte writes)
__host__ __device__ inline int lproj_flat_slice(int K, int TB) {
  const int tile = kTileRows * 2 * K + 2, staged = TB * 64 * 4;
  return ((tile > staged ? tile : staged) + 3) & ~3;
}

template <int DT, int CP, int TB>
__global__ __launch_bounds__(256, 2) void k_lproj_flat(const void* __restrict__ g,
                                                       const int32_t* __restrict__ omega,
                                                       const uint32_t* __restrict__ tile_start,
                                                       float2* __restrict__ gs, const float2* __restrict__ U,
                                                       int rn, int64_t A, int K, int M, int64_t ntiles,
                                                       FusedNext fz) {
  typedef typename BufPair<DT>::type Raw;
  constexpr int W = 4, T = 64 * W;
  constexpr int kPiece = (int)sizeof(Raw);                     // bytes of G per lane and load (2 elements)
  constexpr int kLoadEvery = (CP - 1) / (TB - 1) >= 2 ? 2 : 1; // row pairs of the first stage per load of the next tile
  static_assert((TB - 1) * kLoadEvery < CP, "the first stage issues all TB loads");
  extern __shared__ float smem[];
  const int stride = 2 * K;                                    // floats per LDS row; K is odd
  const int slice = lproj_flat_slice(K, TB);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* sX = smem + wave * slice;
  float2* sF = reinterpret_cast<float2*>(smem + W * slice);
  const int J = (K + 1) >> 1;
  const int N2 = 2 * M;                                        // <= 32: one column tile
  const int ld = 16;
  for (int e = lane; e < slice; e += 64) sX[e] = 0.f;          // pads stay finite
  stage_factor_table<true>(sF, U, rn, K, M, 2 * J, ld, tid, T);
  __syncthreads();                                             // the only workgroup barrier
  const int col = lane & 31, half = lane >> 5, part = col & 1;
  float2 creg[CP];                                             // first-stage coefficients, one pair per row pair
  {
    const float2* fl0 = sF + half * ld + (col >> 1);
#pragma unroll
    for (int j = 0; j < CP; ++j)
      creg[j] = j < J ? column_coef(fl0[2 * j * ld], part) : make_float2(0.f, 0.f);
  }
  float sgn = part ? 1.f : -1.f;                               // (Y J): re column <- -im, im column <- re
  asm volatile("" : "+v"(sgn));                                // (kept a multiplication: it takes the lane swap as its operand modifier)

  const uint32_t tile_elems = (uint32_t)(kTileRows * K);
  const uint32_t tile_bytes = tile_elems * (uint32_t)(kPiece / 2);
  const int S = fz.S;
  const int nslabs = (int)(ntiles / S);                        // whole slabs (host); tile counts fit 32 bits
  const int nw = (int)gridDim.x * W;
  int slab = (int)blockIdx.x * W + wave;
  int ts = 0;
  if (slab >= nslabs) return;
  auto advance = [&](int& sl, int& t) {
    if (t + 1 < S) { t += 1; } else { t = 0; sl += nw; }
  };
  // loop-invariant lane addresses
  const int voff_g = lane * kPiece;                            // into the tile, bytes
  float* sW = sX + lane * 4;                                   // commit: piece i goes to sW + i * 256
  const float* xa = sX + col * stride + 2 * half;              // matrix-core A operand: own row, own half of a pair
  const bool full_out = fz.M2 == 32 && N2 == 32;
  const uint32_t voff_out = (uint32_t)(4 * half * N2 + col);

  Raw raw[TB];
  int32_t my_om = 0;
  // bytes of the tile from the first piece of every group of 4 loads on (scalar registers: a
  // saturating subtraction inside the loop would be done by the vector ALU)
  constexpr int kGroups = (TB + 3) / 4;
  uint32_t rest[kGroups];
#pragma unroll
  for (int k = 0; k < kGroups; ++k) {
    const uint32_t done = (uint32_t)(k * 4 * 64 * kPiece);
    rest[k] = __builtin_amdgcn_readfirstlane(tile_bytes > done ? tile_bytes - done : 0u);
  }
  // piece i of tile t -> raw[i]; the first 64 support entries of a tile -> my_om.  Nothing here uses
  // the vector ALU.  (A descriptor per 4 pieces: immediate offsets reach 4 KB.)
  auto issue_piece = [&](int t, int i) {
    const char* tb = reinterpret_cast<const char*>(g) + (int64_t)t * (int64_t)tile_bytes;
    const int k = i / 4;
    const __amdgpu_buffer_rsrc_t r = raw_buffer(tb + (uint32_t)(k * 4 * 64 * kPiece), rest[k]);
    raw[i] = BufPair<DT>::load(r, voff_g + (i - 4 * k) * 64 * kPiece);
  };
  auto issue_support = [&](uint32_t j0, uint32_t j1) {
    const uint32_t cnt = j1 - j0;                              // (s_min_u32: scalar)
    const __amdgpu_buffer_rsrc_t ro = raw_buffer(omega + j0, (cnt < 64u ? cnt : 64u) * 4u);
    my_om = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(ro, lane * 4, 0, 0);
  };
  const uint32_t vzero = (uint32_t)opaque_zero();
  auto range_of = [&](int t, uint32_t& j0, uint32_t& j1) {   // per-lane loads (scalar base), made scalar when used
    const uint32_t* tsb = tile_start + t;
    j0 = tsb[vzero];
    j1 = tsb[vzero + 1];
  };
  int tile = slab * S;
  int nslab = slab;
  int nts = ts;
  advance(nslab, nts);
  bool have_next = nslab < nslabs;
  int nxt = have_next ? nslab * S + nts : tile;            // past the end: reload the current tile (unused)
  uint32_t cj0v, cj1v, nj0v, nj1v;
  range_of(tile, cj0v, cj1v);
  range_of(nxt, nj0v, nj1v);
  uint32_t cj0 = __builtin_amdgcn_readfirstlane(cj0v), cj1 = __builtin_amdgcn_readfirstlane(cj1v);
#pragma unroll
  for (int i = 0; i < TB; ++i) issue_piece(tile, i);
  issue_support(cj0, cj1);
  v16f acc2;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc2[r] = 0.f;
  // D2 of a complete slab -> out[slab, m2, c].  Issued at the start of the NEXT tile's staging phase,
  // not after the last matrix-core instruction: the wait that opens a tile covers every vector-memory
  // operation before it, and stores issued just before it would be waited for in full.
  auto store_slab = [&](int sl) {
    float* ob = fz.out + (size_t)sl * fz.M2 * N2;
    if (full_out) {                                            // scalar row bases + one invariant lane offset
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float* orow = ob + ((r & 3) + 8 * (r >> 2)) * N2;
        orow[voff_out] = acc2[r];
        acc2[r] = 0.f;
      }
    } else {                                                   // narrower ranks: guarded, addresses made on the spot
      int lane_now = lane;                                     // (opaque: nothing of this is kept in registers across tiles)
      asm volatile("" : "+v"(lane_now));
      const int c2 = lane_now & 31, h2 = lane_now >> 5;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m2 = d_row(r, h2);
        if (m2 < fz.M2 && c2 < N2) ob[m2 * N2 + c2] = acc2[r];
        acc2[r] = 0.f;
      }
    }
  };
  bool pending = false;
  int pending_slab = 0;
  while (true) {
    const uint32_t e_base = (uint32_t)tile * tile_elems;        // I < 2^31
    wave_sync();                                               // previous tile's LDS reads are done
    asm volatile("" : "+v"(my_om));
#pragma unroll
    for (int i = 0; i < TB; ++i) asm volatile("" : "+v"(raw[i]));   // one wait for the whole batch
#pragma unroll
    for (int i = 0; i < TB; ++i) BufPair<DT>::commit(sW + i * 256, raw[i]);
    __builtin_amdgcn_sched_barrier(0);                         // (loads moved above these writes would need register copies)
    if (pending) store_slab(pending_slab);
    // second-stage factor operands of this tile: small, cache-resident; before the next tile's loads
    float2 f2s[16];
    {
      const float4* fp = reinterpret_cast<const float4*>(fz.fpad) + (size_t)ts * 8 * 64;
#pragma unroll
      for (int rp = 0; rp < 8; ++rp) {
        const float4 f = fp[rp * 64 + lane];
        f2s[2 * rp] = make_float2(f.x, f.y);
        f2s[2 * rp + 1] = make_float2(f.z, f.w);
      }
    }
    const int32_t cur_om = my_om;
    int nnslab = nslab;
    int nnts = nts;
    advance(nnslab, nnts);
    const bool have_nn = have_next && nnslab < nslabs;
    const int nn = have_nn ? nnslab * S + nnts : nxt;
    const uint32_t nj0 = __builtin_amdgcn_readfirstlane(nj0v), nj1 = __builtin_amdgcn_readfirstlane(nj1v);
    wave_sync();
    // Sparse(G, Omega) of this tile: hand the values over, then remove them
    {
      float2* gsb = gs + cj0;
      const uint32_t cnt = cj1 - cj0;
      if ((uint32_t)lane < cnt) {
        const uint32_t e = (uint32_t)cur_om - e_base;            // the entry lies in this tile
        float2* p = reinterpret_cast<float2*>(sX + 2 * e);
        gsb[lane] = *p;
        *p = make_float2(0.f, 0.f);
      }
      if (cnt > 64u)
        for (uint32_t j = 64u + lane; j < cnt; j += 64) {
          const uint32_t e = (uint32_t)omega[cj0 + j] - e_base;
          float2* p = reinterpret_cast<float2*>(sX + 2 * e);
          gsb[j] = *p;
          *p = make_float2(0.f, 0.f);
        }
    }
    wave_sync();
    // ---- the 32 rows through the matrix cores ----
    __builtin_amdgcn_s_setprio(1);
    v16f acc;
    {
      // CP row pairs, straight-line, A operands fetched kJUnroll pairs ahead at constant offsets.  Pairs
      // past J meet zero coefficients; what they read lies in the wavefront's own slice (the host
      // checks 62 K + 4 CP <= TB x 256) and is tile data or zeros, so it is finite.
      float2 a2[kJUnroll];
#pragma unroll
      for (int u = 0; u < kJUnroll; ++u) a2[u] = *reinterpret_cast<const float2*>(xa + 4 * u);
#pragma unroll
      for (int jj = 0; jj < CP; ++jj) {
        const float2 a = a2[jj % kJUnroll];
        if (jj + kJUnroll < CP) a2[jj % kJUnroll] = *reinterpret_cast<const float2*>(xa + 4 * (jj + kJUnroll));
        if (jj == 0) {
          v16f zero;
#pragma unroll
          for (int r = 0; r < 16; ++r) zero[r] = 0.f;
          acc = mfma32(a.x, creg[0].x, zero);
        } else {
          acc = mfma32(a.x, creg[jj].x, acc);
        }
        acc = mfma32(a.y, creg[jj].y, acc);
        // The next tile's loads, one per row pair: a load instruction waits at issue until the memory
        // pipeline takes it (at the rate memory delivers when every wavefront streams), and here that
        // wait lies under the matrix-core instructions instead of in front of them.
        if (jj % kLoadEvery == 0 && jj / kLoadEvery < TB) {
          __builtin_amdgcn_sched_barrier(0);
          issue_piece(nxt, jj / kLoadEvery);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    issue_support(nj0, nj1);
    uint32_t nnj0v, nnj1v;
    range_of(nn, nnj0v, nnj1v);
    asm volatile("" : "+v"(f2s[0].x));                         // the factor operands are claimed here
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float y = acc[r];
      const float sw = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(y), 0xB1, 0xF, 0xF, true));
      const float yj = sw * sgn;
      acc2 = mfma32(f2s[r].x, y, acc2);
      acc2 = mfma32(f2s[r].y, yj, acc2);
    }
    const bool slab_done = ts == S - 1;
    const int done_slab = slab;
    __builtin_amdgcn_s_setprio(0);
    pending = slab_done;
    pending_slab = done_slab;
    if (!have_next) break;
    tile = nxt;
    slab = nslab;
    ts = nts;
    nxt = nn;
    nslab = nnslab;
    nts = nnts;
    have_next = have_nn;
    cj0 = nj0;
    cj1 = nj1;
    nj0v = nnj0v;
    nj1v = nnj1v;
  }
  if (pending) store_slab(pending_slab);
}

// k_lupdate: tile = c_alpha * (z x_N U) + c_lambda * scatter(N_S);  W <- decay * W + tile,
// with c_alpha = -lr alpha, c_lambda = -lr lambda, decay = 1 - lr wd (Algorithm 1: "Reconstruct
// low-rank part", "Add scaled sparse tensor", weight update; AdamUpdate on the sparse values
// as in the appendix algorithm "Adam with low-rank tensor decomposition").
// The rows of z are read straight into matrix-core operand registers: lane (row, half) keeps
// elements k = half JT .. half JT + JT - 1 of its row (JT = a power of two >= K / 2, zero beyond
// K), so step (j, part) pairs element j (lanes 0..31) with element JT + j (lanes 32..63).
constexpr int kUpdPrefetch = 17;          // complex64 pairs of W per lane kept in flight during the MFMA phase (the
                                          // most; narrower last modes use 9 or 5: a tile of M-wide rows has M / 4)

template <int WDT, int W, int NTB, int JT, int UP>
__global__ __launch_bounds__(64 * W, 2) void k_lupdate(const float* __restrict__ z,
                                                       const float2* __restrict__ U, int64_t A, int K,
                                                       int M, int64_t ntiles, void* __restrict__ w,
                                                       float decay, float c_alpha, SparseAdam sp) {
  typedef WStore<WDT> WS;
  typedef typename WS::raw wraw;
  constexpr int kPre = WS::kElems == 2 ? UP : (UP + 1) / 2;   // 16-byte pieces of the W tile per lane in flight
  constexpr int T = 64 * W;
  extern __shared__ float smem[];
  const int N2 = 2 * M;
  const int NT = (N2 + 31) >> 5;
  const int ld = 16 * NT;
  const int slice = (kTileRows * N2 + 3) & ~3;                 // floats per wavefront: flat image of its W tile
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // in a scalar register: tile bookkeeping stays scalar
  float* sD = smem + wave * slice;
  float2* sF = reinterpret_cast<float2*>(smem + W * slice);
  stage_factor_table<false>(sF, U, K, K, M, 2 * JT, ld, tid, T, c_alpha);   // the update's scale rides in the table
  __syncthreads();                                             // the only workgroup barrier
  // a lone last complex column (half-spectrum modes have 2^m + 1 entries) does not get a 32-column
  // matrix-core tile of its own: it is expanded with vector arithmetic (see k_lupdate_fused)
  const bool vtail = (N2 & 31) == 2;
  const int NTm = vtail ? NT - 1 : NT;

  const int64_t Iw = A * M;                                    // complex elements of W
  const int tile_w = kTileRows * M;
  const int64_t step = (int64_t)gridDim.x * W;
  int64_t tile = (int64_t)blockIdx.x * W + wave;
  if (tile >= ntiles) return;
  const float2* zall = reinterpret_cast<const float2*>(z);

  float2 zreg[JT];
  int32_t my_om = -1;
  float2 my_g = make_float2(0.f, 0.f), my_m = make_float2(0.f, 0.f);
  float my_v = 0.f;
  // operand rows and sparse state of tile `t` (support range [j0, j1))
  auto issue_small = [&](int64_t t, uint32_t j0, uint32_t j1) {
    const int col = lane & 31, half = lane >> 5;
    const int64_t grow = t * kTileRows + col;
    const float2* zr = zall + grow * K + half * JT;
#pragma unroll
    for (int j = 0; j < JT; ++j) {
      zreg[j] = make_float2(0.f, 0.f);
      if (grow < A && half * JT + j < K) zreg[j] = zr[j];
    }
    my_om = -1;
    if (j0 + lane < j1) {
      my_om = sp.omega[j0 + lane];
      my_g = sp.gs[j0 + lane];
      my_m = sp.ms[j0 + lane];
      my_v = sp.vs[j0 + lane];
    }
  };

  const int vzero = opaque_zero();                             // see k_lproj
  int64_t nxt = tile + step;
  uint32_t cj0 = sp.tile_start[tile + vzero], cj1 = sp.tile_start[tile + 1 + vzero];
  uint32_t nj0 = 0, nj1 = 0;
  if (nxt < ntiles) {
    nj0 = sp.tile_start[nxt + vzero];
    nj1 = sp.tile_start[nxt + 1 + vzero];
  }
  // Every wait for loads sits at ONE point per tile (claim_loads, before the stream-out), where the
  // only younger memory operations are loads that are needed right after anyway.  Loads retire
  // in order, so a wait anywhere else would also wait for stores or loads issued after it.
  auto claim_small = [&]() {
#pragma unroll
    for (int j = 0; j < JT; ++j) asm volatile("" : "+v"(zreg[j].x), "+v"(zreg[j].y));
    asm volatile("" : "+v"(my_om), "+v"(my_g.x), "+v"(my_g.y), "+v"(my_m.x), "+v"(my_m.y), "+v"(my_v));
  };
  issue_small(tile, cj0, cj1);
  claim_small();
  while (true) {
    int lane_now = lane;                                       // opaque per-tile copy (see k_lproj)
    asm volatile("" : "+v"(lane_now));
    const int col = lane_now & 31, half = lane_now >> 5;
    const float2* fl = sF + half * JT * ld + (col >> 1);
    const int part = col & 1;
    const int64_t w_base = tile * tile_w;                      // complex index of the tile in W
    const int n_w = (int)((Iw - w_base) < tile_w ? (Iw - w_base) : tile_w);
    wraw* w4 = WS::tile(w, w_base);                            // 16-byte aligned: a tile holds 32 M elements
    const int n4 = n_w / WS::kElems;                           // whole 16-byte pieces
    // ---- what was fetched one tile ago moves out of the prefetch registers; the next tile's small
    //      loads and this tile's W pieces go in flight ----
    float2 zcur[JT];
#pragma unroll
    for (int j = 0; j < JT; ++j) zcur[j] = zreg[j];
    const int32_t c_om = my_om;
    const float2 c_g = my_g, c_m = my_m;
    const float c_v = my_v;
    const int64_t nn = nxt + step;
    uint32_t nnj0 = 0, nnj1 = 0;
    if (nxt < ntiles) {
      issue_small(nxt, nj0, nj1);
      if (nn < ntiles) {
        nnj0 = sp.tile_start[nn + vzero];
        nnj1 = sp.tile_start[nn + 1 + vzero];
      }
    }
    wraw wpre[kPre];                                  // unconditional loads, clamped onto the last
#pragma unroll                                                 // piece (the host keeps n4 >= 1 for every tile)
    for (int i = 0; i < kPre; ++i) {
      const int q = lane_now + i * 64;
      wpre[i] = nt_load(&w4[q < n4 ? q : n4 - 1]);
    }
    wave_sync();                                               // previous tile's LDS reads are done
    // ---- expand the 32 rows: sD[row, c] = sum_k (c_alpha U)[c, k] z[row, k], NTB column tiles at a time ----
    auto block = [&](int nt0, auto ntile_count) {
      constexpr int N = decltype(ntile_count)::value;
      v16f acc[N];
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
      const float2* fb = fl + 16 * nt0;
#pragma unroll
      for (int j = 0; j < JT; ++j) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const float2 b2 = column_coef(fb[j * ld + 16 * i], part);
          acc[i] = mfma32(zcur[j].x, b2.x, acc[i]);
          acc[i] = mfma32(zcur[j].y, b2.y, acc[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int c = 32 * (nt0 + i) + col;
        if (c < N2) {
#pragma unroll
          for (int r = 0; r < 16; ++r) sD[d_row(r, half) * N2 + c] = acc[i][r];
        }
      }
    };
    {
      int nt0 = 0;
      for (; nt0 + NTB <= NTm; nt0 += NTB) block(nt0, std::integral_constant<int, NTB>());
      if (NTB > 1)
        for (; nt0 < NTm; ++nt0) block(nt0, std::integral_constant<int, 1>());
    }
    if (vtail) {                                               // the last complex column, without the matrix cores
      const float2* ft = sF + half * JT * ld + (M - 1);
      float pre = 0.f, pim = 0.f;
#pragma unroll
      for (int jj = 0; jj < JT; ++jj) {
        const float2 cf = ft[jj * ld];
        pre += zcur[jj].x * cf.x - zcur[jj].y * cf.y;
        pim += zcur[jj].x * cf.y + zcur[jj].y * cf.x;
      }
      pre += __shfl_xor(pre, 32, 64);
      pim += __shfl_xor(pim, 32, 64);
      if (half == 0) *reinterpret_cast<float2*>(&sD[col * N2 + N2 - 2]) = make_float2(pre, pim);
    }
    wave_sync();
    // ---- AdamUpdate on the sparse values that live in this tile; add lambda N_S into the tile ----
    if (cj0 + lane < cj1) sparse_adam_entry(sp, cj0 + lane, c_om, c_g, c_m, c_v, w_base, sD);
    if (cj1 - cj0 > 64u)                                       // rare: more than 64 entries in one tile
      for (uint32_t j = cj0 + 64u + lane; j < cj1; j += 64)
        sparse_adam_entry(sp, j, sp.omega[j], sp.gs[j], sp.ms[j], sp.vs[j], w_base, sD);
    wave_sync();
    // ---- stream the tile into W ----
    claim_small();
#pragma unroll
    for (int i = 0; i < kPre; ++i) claim_raw(wpre[i]);
    const int nfull = n4 >> 6;                                 // pieces every lane owns: no per-lane branch
#pragma unroll
    for (int i = 0; i < kPre; ++i) {
      const int q = lane_now + i * 64;
      if (i < nfull || q < n4) nt_store(&w4[q], WS::apply(wpre[i], sD, q, decay));
    }
    for (int q = lane + kPre * 64; q < n4; q += 64) w4[q] = WS::apply(w4[q], sD, q, decay);
    {                                                          // elements past the last whole piece
      const int e = n4 * WS::kElems + lane;
      if (e < n_w) WS::apply_one(w, w_base + e, sD + 2 * e, decay);
    }
    if (nxt >= ntiles) break;
    tile = nxt;
    nxt = nn;
    cj0 = nj0;
    cj1 = nj1;
    nj0 = nnj0;
    nj1 = nnj1;
  }
}

// k_lupdate_fused: k_lupdate with the reconstruction stage of mode N-1 (extent 32 S, rank K2 <= 32)
// in front of it, so the tensor between the two stages never exists.  A wavefront walks whole
// slabs; per tile (32 rows i2 of the slab):
//   stage A   D'[(m3, p), i2] = sum_m2 Y1[m2, m3] U2[i2, m2]            (rows = interleaved (m3, p))
//             A operand: lane (rho = 2 m3 + p, half) holds Y1[2 jj + half][m3] (parts chosen per p and
//             per factor part: re(u y) = ur yr - ui yi, im(u y) = ur yi + ui yr),
//             B operand: U2[i2, 2 jj + half] from the packed copy `ut` (two steps per 16-byte load);
//   stage B   the accumulator registers of D' ARE the operand rows of the last-mode expansion: in lane
//             (i2, half) registers (2 u, 2 u + 1) hold (re, im) of element k = (u & 1) + 4 (u >> 1) + 2 half
//             of row i2, so step (u, part) pairs elements k(u, 0) and k(u, 1) and the coefficient
//             table is read at those rows.  Everything after that is k_lupdate.
struct FusedPrev {
  const float2* y1;     // input of the fused stage, (slabs, K2, K) complex
  const float2* ut;     // U^(N-1)[i2, m2], zero for m2 >= K2, in operand order (k_pack_fused_factor)
  int S;                // tiles per slab
  int K2;               // rank of mode N-1
};

template <int WDT, int W, int MS, int JT2, int UP>
__global__ __launch_bounds__(64 * W, 2) void k_lupdate_fused(const float2* __restrict__ U, int64_t A, int K,
                                                             int M, int64_t ntiles, void* __restrict__ w,
                                                             float decay, float c_alpha, SparseAdam sp,
                                                             FusedPrev fz) {
  typedef WStore<WDT> WS;
  typedef typename WS::raw wraw;
  constexpr int kPre = WS::kElems == 2 ? UP : (UP + 1) / 2;   // 16-byte pieces of the W tile per lane in flight
  constexpr int T = 64 * W;
  extern __shared__ float smem[];
  // MS > 0: the extent of the last mode is the compile-time constant MS (the host passes M == MS): stage B
  // then runs without a single vector-ALU instruction between its matrix instructions (see below).
  const int N2 = MS > 0 ? 2 * MS : 2 * M;
  const int NT = (N2 + 31) >> 5;
  const int ld = 16 * NT;
  const int slice = (kTileRows * N2 + 3) & ~3;                 // floats per wavefront: flat image of its W tile
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* sD = smem + wave * slice;
  float2* sF = reinterpret_cast<float2*>(smem + W * slice);
  stage_factor_table<false>(sF, U, K, K, M, 16, ld, tid, T, c_alpha);   // 16 rows: K <= 16 here; scaled by c_alpha
  __syncthreads();                                             // the only workgroup barrier
  // A half-spectrum last mode has 2^m + 1 entries: its last complex column would occupy a whole
  // 32-column matrix-core tile on its own.  That column is expanded with ordinary arithmetic
  // instead: each lane holds 8 of the 16 elements of its row (see stage B), multiplies them with
  // the column's coefficients - which do not depend on the tile and stay in registers - and the
  // two halves of the wavefront are added with one lane exchange.
  const bool vtail = (N2 & 31) == 2;
  const int NTm = vtail ? NT - 1 : NT;                         // column tiles that go through the matrix cores
  float2 ctail[8];                                             // (MS > 0: read from the table when used; the registers
#pragma unroll                                                 //  hold the matrix-core coefficients instead)
  for (int u = 0; u < 8; ++u) {
    const int k = (u & 1) + 4 * (u >> 1) + 2 * (lane >> 5);
    ctail[u] = (MS == 0 && vtail) ? sF[k * ld + (M - 1)] : make_float2(0.f, 0.f);
  }

  // MS > 0: the stage-B coefficients of every column tile, already in the form the lane's column needs
  // (they do not depend on the tile), in registers for the whole kernel.
  constexpr int kNTmS = MS > 0 ? ((2 * MS) & 31) == 2 ? (2 * MS + 31) / 32 - 1 : (2 * MS + 31) / 32 : 1;
  float2 cregB[kNTmS][8];
  if constexpr (MS > 0) {
    const float2* fl0 = sF + (2 * (lane >> 5)) * ld + ((lane & 31) >> 1);
#pragma unroll
    for (int i = 0; i < kNTmS; ++i)
#pragma unroll
      for (int u = 0; u < 8; ++u)
        cregB[i][u] = column_coef(fl0[((u & 1) + 4 * (u >> 1)) * ld + 16 * i], lane & 1);
  }

  const int64_t Iw = A * M;
  const int tile_w = kTileRows * M;
  const int S = fz.S;
  const int64_t nslabs = ntiles / S;                           // A = slabs * 32 S exactly
  const int64_t nw = (int64_t)gridDim.x * W;
  int64_t slab = (int64_t)blockIdx.x * W + wave;
  int ts = 0;
  if (slab >= nslabs) return;
  auto advance = [&](int64_t& sl, int& t) {
    if (t + 1 < S) { t += 1; } else { t = 0; sl += nw; }
  };

  int32_t my_om = -1;
  float2 my_g = make_float2(0.f, 0.f), my_m = make_float2(0.f, 0.f);
  float my_v = 0.f;
  const int om_last = sp.k_last;
  // sparse state of a tile with support range [j0, j1): fetched one tile ahead; unconditional loads
  // (lanes without an entry read a clamped, valid position and ignore it)
  auto issue_sparse = [&](uint32_t j0, uint32_t j1) {
    const uint32_t j = j0 + lane;
    const uint32_t jc = j < j1 ? j : (uint32_t)om_last;
    my_om = j < j1 ? sp.omega[jc] : -1;
    my_g = sp.gs[jc];
    my_m = sp.ms[jc];
    my_v = sp.vs[jc];
  };
  auto claim_sparse = [&]() {
    asm volatile("" : "+v"(my_om), "+v"(my_g.x), "+v"(my_g.y), "+v"(my_m.x), "+v"(my_m.y), "+v"(my_v));
  };

  const int vzero = opaque_zero();
  // W goes through buffer descriptors (one per 4 pieces), range-checked by the hardware: no clamps
  // and no lane masks in the streaming phase.  Bytes of a tile from the first piece of each group on:
  constexpr int kWGroups = (kPre + 3) / 4;
  const uint32_t w_tile_bytes = (uint32_t)tile_w * (uint32_t)(16 / WS::kElems);
  uint32_t w_rest[kWGroups];
#pragma unroll
  for (int k = 0; k < kWGroups; ++k) {
    const uint32_t done = (uint32_t)(k * 4 * 64 * 16);
    w_rest[k] = __builtin_amdgcn_readfirstlane(w_tile_bytes > done ? w_tile_bytes - done : 0u);
  }
  const int voff_w = lane * 16;
  int64_t tile = slab * S;
  int64_t nslab = slab;
  int nts = ts;
  advance(nslab, nts);
  bool have_next = nslab < nslabs;
  int64_t nxt = have_next ? nslab * S + nts : tile;
  uint32_t cj0 = sp.tile_start[tile + vzero], cj1 = sp.tile_start[tile + 1 + vzero];
  uint32_t nj0 = sp.tile_start[nxt + vzero], nj1 = sp.tile_start[nxt + 1 + vzero];
  issue_sparse(cj0, cj1);
  claim_sparse();
  // Stage-A operand rows (the slab's Y1) stay in registers for all S tiles of a slab.  Those of the NEXT slab
  // are requested right after stage A of a slab's last tile, when the registers have just been used
  // for the last time: they then have a whole stage B and W phase to arrive.  Unconditional
  // loads with clamped indices: clamped rows / columns meet zero coefficients.
  float2 y1[JT2];
  auto fetch_y1 = [&](int64_t sl, int ln) {
    const int c2 = ln & 31, h2 = ln >> 5;
    const int m3 = (c2 >> 1) < K ? (c2 >> 1) : K - 1;
    const float2* yp = fz.y1 + sl * fz.K2 * K + m3;
#pragma unroll
    for (int jj = 0; jj < JT2; ++jj) {
      const int m2 = 2 * jj + h2;
      y1[jj] = yp[(m2 < fz.K2 ? m2 : fz.K2 - 1) * K];
    }
  };
  fetch_y1(slab, lane);
  while (true) {
    int lane_now = lane;                                       // opaque per-tile copy (see k_lproj)
    asm volatile("" : "+v"(lane_now));
    const int col = lane_now & 31, half = lane_now >> 5;
    const int part = col & 1;
    const int64_t w_base = tile * tile_w;
    const int n_w = (int)((Iw - w_base) < tile_w ? (Iw - w_base) : tile_w);
    wraw* w4 = WS::tile(w, w_base);
    const int n4 = n_w / WS::kElems;                           // tiles are whole here: 32 M elements, a multiple of 4
    const int32_t c_om = my_om;
    const float2 c_g = my_g, c_m = my_m;
    const float c_v = my_v;
    // ---- this tile's 32 columns of the factor copy (small, cache-resident), issued BEFORE the W pieces so
    //      that waiting for them leaves those in flight ----
    float2 u2[JT2];
    {
      const float4* up = reinterpret_cast<const float4*>(fz.ut) + (size_t)ts * 8 * 64 + lane_now;
#pragma unroll
      for (int jp = 0; jp < JT2 / 2; ++jp) {                   // two operand rows per 16-byte load
        const float4 f = up[jp * 64];
        u2[2 * jp] = make_float2(f.x, f.y);
        u2[2 * jp + 1] = make_float2(f.z, f.w);
      }
    }
    // ---- this tile's W pieces go in flight ----
    wraw wpre[kPre];
    const char* w_tile = reinterpret_cast<const char*>(w4);
#pragma unroll
    for (int k = 0; k < kWGroups; ++k) {                       // a descriptor per 4 pieces: immediates reach 4 KB
      const __amdgpu_buffer_rsrc_t r = raw_buffer(w_tile + k * 4 * 64 * 16, w_rest[k]);
#pragma unroll
      for (int i = 4 * k; i < 4 * k + 4 && i < kPre; ++i) buffer_piece_load(wpre[i], r, voff_w + (i - 4 * k) * 64 * 16);
    }
    // The stage-A operands are claimed here: the asm statements pin every load above them (memory
    // clobber) and every use below them, so the scheduler cannot interleave load - wait - MFMA.
#pragma unroll
    for (int jj = 0; jj < JT2; ++jj)
      asm volatile("" : "+v"(y1[jj].x), "+v"(y1[jj].y), "+v"(u2[jj].x), "+v"(u2[jj].y) : : "memory");
    // ---- stage A: D' = rows of the mode-(N-1) expansion for the 32 rows of the tile ----
    v16f dz;
#pragma unroll
    for (int r = 0; r < 16; ++r) dz[r] = 0.f;
    if (ts == 0) {
      // (wave-uniform) first tile of a slab: the rows just claimed become the two A operands of the lane's
      // row (rho = 2 m3 + p): re(u y) = ur yr - ui yi, im(u y) = ur yi + ui yr; once per slab, not per tile
#pragma unroll
      for (int jj = 0; jj < JT2; ++jj) {
        const float2 y = y1[jj];
        y1[jj].x = part ? y.y : y.x;
        y1[jj].y = part ? y.x : -y.y;
      }
    }
#pragma unroll
    for (int jj = 0; jj < JT2; ++jj) {
      dz = mfma32(y1[jj].x, u2[jj].x, dz);
      dz = mfma32(y1[jj].y, u2[jj].y, dz);
    }
    if (nts == 0 && have_next) fetch_y1(nslab, lane_now);      // (wave-uniform) the next tile opens a new slab
    // ---- the next tile's sparse state goes in flight ----
    int64_t nnslab = nslab;
    int nnts = nts;
    advance(nnslab, nnts);
    const bool have_nn = have_next && nnslab < nslabs;
    const int64_t nn = have_nn ? nnslab * S + nnts : nxt;
    issue_sparse(nj0, nj1);
    const uint32_t nnj0 = sp.tile_start[nn + vzero], nnj1 = sp.tile_start[nn + 1 + vzero];
    wave_sync();                                               // previous tile's LDS reads are done
    // ---- stage B: expand the last mode: sD[row, c] = sum_k (c_alpha U)[c, k] ..., NTB column tiles at a time ----
    const float2* fl = sF + (2 * half) * ld + (col >> 1);      // row k(u, half) = (u & 1) + 4 (u >> 1) + 2 half
    if constexpr (MS > 0) {
      // Straight-line: 16 matrix instructions per column tile with coefficients from registers, then the tile's
      // 16 result rows written at constant offsets from one lane address.  (A vector-ALU instruction between two fp32 matrix instructions waits for the matrix
      // pipe: selects, zeroing and register copies in this stage cost more than its matrix work.)
      constexpr int N2s = 2 * MS;
      float* sDl = sD + (4 * half) * N2s + col;
      auto chain = [&](int i) -> v16f {
        v16f zero;
#pragma unroll
        for (int r = 0; r < 16; ++r) zero[r] = 0.f;
        v16f acc = mfma32(dz[0], cregB[i][0].x, zero);
        acc = mfma32(dz[1], cregB[i][0].y, acc);
#pragma unroll
        for (int u = 1; u < 8; ++u) {
          acc = mfma32(dz[2 * u], cregB[i][u].x, acc);
          acc = mfma32(dz[2 * u + 1], cregB[i][u].y, acc);
        }
        return acc;
      };
      auto put = [&](const v16f& acc, int i) {
        if (32 * (i + 1) <= N2s || 32 * i + col < N2s) {
#pragma unroll
          for (int r = 0; r < 16; ++r) sDl[((r & 3) + 8 * (r >> 2)) * N2s + 32 * i] = acc[r];
        }
      };
#pragma unroll
      for (int i = 0; i < kNTmS; ++i) put(chain(i), i);
    } else {
      // one column tile at a time, its 8 coefficient pairs fetched while the previous tile is in the
      // matrix cores (the last tile re-reads itself)
      float2 cf[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) cf[u] = fl[((u & 1) + 4 * (u >> 1)) * ld];
      for (int nt0 = 0; nt0 < NTm; ++nt0) {
        float2 cn[8];
        const float2* fn = fl + 16 * (nt0 + 1 < NTm ? nt0 + 1 : nt0);
#pragma unroll
        for (int u = 0; u < 8; ++u) cn[u] = fn[((u & 1) + 4 * (u >> 1)) * ld];
        v16f acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const float2 b2 = column_coef(cf[u], part);
          acc = mfma32(dz[2 * u], b2.x, acc);
          acc = mfma32(dz[2 * u + 1], b2.y, acc);
        }
        const int c = 32 * nt0 + col;
        if (c < N2) {
#pragma unroll
          for (int r = 0; r < 16; ++r) sD[d_row(r, half) * N2 + c] = acc[r];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) cf[u] = cn[u];
      }
    }
    if (vtail) {                                               // the last complex column, without the matrix cores
      float pre = 0.f, pim = 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float zr = dz[2 * u], zi = dz[2 * u + 1];
        const float2 ct = MS > 0 ? sF[((u & 1) + 4 * (u >> 1) + 2 * half) * ld + (MS - 1)] : ctail[u];
        pre += zr * ct.x - zi * ct.y;
        pim += zr * ct.y + zi * ct.x;
      }
      pre += __shfl_xor(pre, 32, 64);
      pim += __shfl_xor(pim, 32, 64);
      if (half == 0) *reinterpret_cast<float2*>(&sD[col * N2 + N2 - 2]) = make_float2(pre, pim);
    }
    wave_sync();
    // ---- AdamUpdate on the sparse values that live in this tile; add lambda N_S into the tile ----
    if (cj0 + lane < cj1) sparse_adam_entry(sp, cj0 + lane, c_om, c_g, c_m, c_v, w_base, sD);
    if (cj1 - cj0 > 64u)                                       // rare: more than 64 entries in one tile
      for (uint32_t j = cj0 + 64u + lane; j < cj1; j += 64)
        sparse_adam_entry(sp, j, sp.omega[j], sp.gs[j], sp.ms[j], sp.vs[j], w_base, sD);
    wave_sync();
    // ---- the wait point for everything still in flight, then stream the tile into W ----
    claim_sparse();
#pragma unroll
    for (int i = 0; i < kPre; ++i) claim_raw(wpre[i]);
#pragma unroll
    for (int k = 0; k < kWGroups; ++k) {                       // (pieces past the tile's end are dropped by the range check)
      const __amdgpu_buffer_rsrc_t r = raw_buffer(w_tile + k * 4 * 64 * 16, w_rest[k]);
#pragma unroll
      for (int i = 4 * k; i < 4 * k + 4 && i < kPre; ++i) {
        const int q = lane_now + i * 64;                       // (the LDS read stays inside the tile)
        buffer_piece_store(WS::apply(wpre[i], sD, q < n4 ? q : n4 - 1, decay), r, voff_w + (i - 4 * k) * 64 * 16);
      }
    }
    for (int q = lane + kPre * 64; q < n4; q += 64) w4[q] = WS::apply(w4[q], sD, q, decay);
    if (!have_next) break;
    tile = nxt;
    slab = nslab;
    ts = nts;
    nxt = nn;
    nslab = nnslab;
    nts = nnts;
    have_next = have_nn;
    cj0 = nj0;
    cj1 = nj1;
    nj0 = nnj0;
    nj1 = nnj1;
  }
}

// Kernel-ready copies of the mode-(N-1) factor for the fused stages:
//   fpad = conj(U[i2, m2]) (m2 < r, else 0; 32 columns), tile by tile in matrix-core operand order
//                                                               -> second compression stage in k_lproj
//   ut   = U[i2, m2] (m2 < r, else 0; 32 columns), tile by tile in matrix-core operand order
//                                                               -> first reconstruction stage in k_lupdate_fused
__global__ void k_pack_fused_factor(const float2* __restrict__ U, int I2, int r, float2* __restrict__ fpad,
                                    float2* __restrict__ ut) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= I2 * 32) return;
  const int i2 = e >> 5, m2 = e & 31;
  const float2 u = m2 < r ? U[(int64_t)i2 * r + m2] : make_float2(0.f, 0.f);
  // fpad in the order the second compression stage consumes it: tile ts = i2 / 32, row i2 % 32 =
  // d_row(rr, half), lane = 32 half + m2; slot [ts][rr / 2][lane][rr % 2], so that a lane fetches the
  // operands of two accumulator rows with one 16-byte load and a wavefront reads 1 KB contiguous
  const int ts = i2 >> 5, il = i2 & 31;
  const int half = (il >> 2) & 1, rr = (il & 3) + 4 * (il >> 3);
  fpad[(((size_t)ts * 8 + (rr >> 1)) * 64 + 32 * half + m2) * 2 + (rr & 1)] = make_float2(u.x, -u.y);
  // ut in the order the first reconstruction stage consumes it: step jj = m2 / 2 of the lane
  // (i2 % 32, m2 % 2); slot [ts][jj / 2][lane][jj % 2]
  const int jj = m2 >> 1;
  ut[(((size_t)ts * 8 + (jj >> 1)) * 64 + 32 * (m2 & 1) + il) * 2 + (jj & 1)] = u;
}

// tile_start[t] = support entries below tile t, t = 0 .. ntiles (Omega ascending).  Tile t of the tensor cut into
// slabs of `slab_elems` elements and those into S tiles of `tile_elems` (the last one of a slab may be shorter)
// starts at element (t / S) slab_elems + (t % S) tile_elems.  Flat tiles: S = 1, slab_elems = tile_elems.
__global__ void k_tile_offsets(const int32_t* __restrict__ omega, int64_t k, int64_t tile_elems, uint32_t S,
                               int64_t slab_elems, int64_t ntiles, uint32_t* __restrict__ tile_start) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t > ntiles) return;
  const uint32_t sl = (uint32_t)t / S;                          // (tile counts fit 32 bits: I < 2^31)
  const int64_t target = (int64_t)sl * slab_elems + (int64_t)((uint32_t)t - sl * S) * tile_elems;
  int64_t lo = 0, hi = k;                                      // first j in [0, k] with Omega_j >= target
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)omega[mid] < target) lo = mid + 1; else hi = mid;
  }
  tile_start[t] = (uint32_t)lo;
}

int grid_for_tiles(int64_t ntiles, int blocks_per_cu) {
  const int64_t cap = (int64_t)compute_units() * blocks_per_cu;
  return (int)(ntiles < cap ? ntiles : cap);
}

}  // namespace

// ---- host side ---------------------------------------------------------------------------------

size_t lproj_lds_bytes(int W, int K, int M) {
  const int stride = 2 * K + ((K & 1) ? 0 : 2), J = (K + 1) / 2, NT = (2 * M + 31) / 32;
  return (size_t)W * (kTileRows * stride + 2) * 4 + (size_t)2 * J * 16 * NT * 8;
}

int lupdate_jt(int K) {                         // operand-register pairs per lane: power of two >= K / 2
  int jt = 1;
  while (2 * jt < K) jt *= 2;
  return jt;
}

size_t lupdate_lds_bytes(int W, int K, int M) {
  const int NT = (2 * M + 31) / 32;
  return (size_t)W * ((kTileRows * 2 * M + 3) & ~3) * 4 + (size_t)2 * lupdate_jt(K) * 16 * NT * 8;
}

constexpr int kUpdMaxJT = 16;                   // k_lupdate keeps a row of z in registers: rank of the last mode <= 32

// Wavefronts per workgroup for the two last-mode kernels (each wavefront stages its own 32-row
// tile in LDS), or 0 if the shape is outside what they cover.  `Klast` / `rlast` are the extent
// and the rank of the last mode.  Two workgroups per compute unit are preferred.
int fused_max_last_extent() { return 2 * kCoefPairs; }

int choose_tile_waves(int Klast, int rlast, int prefer) {
  if (lupdate_jt(rlast) > kUpdMaxJT) return 0;
  if (Klast < 2) return 0;                      // the tile loaders assume at least one 2-element piece per tile
  if ((int64_t)kTileRows * Klast >= (1 << 17)) return 0;
  const int cand[3] = {4, 2, 1};
  for (int pass = 0; pass < 2; ++pass) {
    const size_t limit = pass == 0 ? kLdsLimit / 2 : kLdsLimit;
    for (int i = 0; i < 3; ++i) {
      const int W = cand[i];
      if (W > prefer) continue;
      if (lproj_lds_bytes(W, Klast, rlast) <= limit && lupdate_lds_bytes(W, rlast, Klast) <= limit) return W;
    }
  }
  return 0;
}

// Launches one of the matrix-core loops over the whole chip (two workgroups of four wavefronts per compute
// unit); returns the real floating-point operations of the launch.
double launch_mfma_probe(hipStream_t s, int kind, int64_t iters, float* sink) {
  const int grid = compute_units() * 2;
  iters = (iters + kProbeUnroll - 1) / kProbeUnroll * kProbeUnroll;
  const double instr = (double)grid * 4.0 * (double)iters * kProbeChains;
  if (kind == 0) {
    k_mfma_probe_f32<<<dim3((unsigned)grid), dim3(256), 0, s>>>(sink, iters, 1.f, 0.5f);
    return instr * 4096.0;                                     // 32 x 32 x 2 multiply-adds
  }
  k_mfma_probe_f64<<<dim3((unsigned)grid), dim3(256), 0, s>>>(sink, iters, 1., 0.5);
  return instr * 2048.0;                                       // 16 x 16 x 4 multiply-adds
}

void launch_tile_offsets(hipStream_t s, const int32_t* omega, int64_t k, int64_t tile_elems, int S,
                         int64_t slab_elems, int64_t ntiles, uint32_t* tile_start) {
  const int64_t n = ntiles + 1;
  k_tile_offsets<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(omega, k, tile_elems, (uint32_t)S,
                                                                        slab_elems, ntiles, tile_start);
}

void launch_pack_fused_factor(hipStream_t s, const float2* U, int I2, int r, float2* fpad, float2* ut) {
  k_pack_fused_factor<<<dim3((unsigned)((I2 * 32 + 255) / 256)), dim3(256), 0, s>>>(U, I2, r, fpad, ut);
}

// `fused_I2` > 0: also contract the next mode (extent fused_I2 = 32 S, rank fused_M2, factor copy
// `fpad`) and write its result to `out` (slabs, fused_M2, M); otherwise `out` is (A, M).
void launch_lproj(hipStream_t s, const void* g, int dtype, const int32_t* omega, const uint32_t* tile_start,
                  float2* gs, const float2* U, int rn, const Stage& st, int W, float2* out, int fused_I2,
                  int fused_M2, const float2* fpad) {
  const int64_t A = st.A;
  const int K = st.K, M = st.M;
  if (A * M <= 0) return;
  if (fused_I2 == 0 && rows_kernel_pays(K, M, A)) return launch_rows(s, g, dtype, omega, tile_start, gs, U, st, out);
  const int64_t ntiles = (A + kTileRows - 1) / kTileRows;
  const size_t lds = lproj_lds_bytes(W, K, M);
  const int NT = (2 * M + 31) / 32;
  const int ntb = NT >= 2 ? 2 : 1;
  const bool fuse = fused_I2 > 0;
  const int S = fuse ? fused_I2 / kTileRows : 1;
  const int64_t nslabs = (ntiles + S - 1) / S;
  const int tb = (K + 3) / 4 <= 5 ? 5 : (K + 3) / 4 <= 9 ? 9 : kTileBatch;   // pieces per lane a tile needs (capped)
  const int64_t ngroups = (nslabs + W - 1) / W;                // workgroups' worth of tile sequences
  dim3 grid(1), block(64 * W);
  float* of = reinterpret_cast<float*>(out);
  const uint32_t magic = magic_for(K);
  FusedNext fz{fpad, of, S, fused_M2};
#define TGRAD_LP_C(DT_, W_, NTB_, F_, Z_, CP_, TB_)                                                      \
  do {                                                                                                   \
    allow_lds(k_lproj<DT_, W_, NTB_, F_, Z_, CP_, TB_>, lds);                                            \
    grid.x = (unsigned)grid_for_tiles(ngroups, resident_blocks(k_lproj<DT_, W_, NTB_, F_, Z_, CP_, TB_>, 64 * W_, lds)); \
    k_lproj<DT_, W_, NTB_, F_, Z_, CP_, TB_><<<grid, block, lds, s>>>(g, omega, tile_start, gs, U, rn,   \
                                                                      A, K, M, magic, ntiles, of, fz);   \
  } while (0)
#define TGRAD_LP(DT_, W_, NTB_, F_) TGRAD_LP_C(DT_, W_, NTB_, F_, false, 1, kTileBatch)
#define TGRAD_LP_FUSED(DT_, F_)                                                                          \
  do {                                                                                                   \
    if ((K + 1) / 2 > kCoefPairsShort) TGRAD_LP_C(DT_, 4, 1, F_, true, kCoefPairs, kTileBatch);          \
    else if (tb == 5) TGRAD_LP_C(DT_, 4, 1, F_, true, kCoefPairsShort, 5);                               \
    else TGRAD_LP_C(DT_, 4, 1, F_, true, kCoefPairsShort, 9);                                            \
  } while (0)
#define TGRAD_LP_F(DT_, W_, NTB_)                                                                        \
  do {                                                                                                   \
    if (K & 1) TGRAD_LP(DT_, W_, NTB_, true); else TGRAD_LP(DT_, W_, NTB_, false);                       \
  } while (0)
#define TGRAD_LP_W(DT_, NTB_)                                                                            \
  do {                                                                                                   \
    if (W == 4 && NTB_ == 1 && tb == 5) {   /* (the shortest rows: rows_kernel_pays) */                  \
      if (K & 1) TGRAD_LP_C(DT_, 4, 1, true, false, 1, 5); else TGRAD_LP_C(DT_, 4, 1, false, false, 1, 5); \
    } else if (W == 4) TGRAD_LP_F(DT_, 4, NTB_); else if (W == 2) TGRAD_LP_F(DT_, 2, NTB_); else TGRAD_LP_F(DT_, 1, NTB_); \
  } while (0)
#define TGRAD_LPF_C(DT_, CP_, TB_)                                                                       \
  do {                                                                                                   \
    const size_t ldsf = (size_t)4 * lproj_flat_slice(K, TB_) * 4 + (size_t)2 * ((K + 1) / 2) * 16 * 8;   \
    allow_lds(k_lproj_flat<DT_, CP_, TB_>, ldsf);                                                        \
    grid.x = (unsigned)grid_for_tiles(ngroups, resident_blocks(k_lproj_flat<DT_, CP_, TB_>, 256, ldsf)); \
    k_lproj_flat<DT_, CP_, TB_><<<grid, block, ldsf, s>>>(g, omega, tile_start, gs, U, rn, A, K, M,      \
                                                          ntiles, fz);                                   \
  } while (0)
#define TGRAD_LPF(DT_)                                                                                   \
  do {                                                                                                   \
    if ((K + 1) / 2 > kCoefPairsShort) TGRAD_LPF_C(DT_, kCoefPairs, kTileBatch);                         \
    else if (tb == 5) TGRAD_LPF_C(DT_, kCoefPairsShort, 5);                                              \
    else TGRAD_LPF_C(DT_, kCoefPairsShort, 9);                                                           \
  } while (0)
  const int cp = (K + 1) / 2 > kCoefPairsShort ? kCoefPairs : kCoefPairsShort;
  if (fuse && (K & 1) && tb * 64 >= 16 * K && 62 * K + 4 * cp <= tb * 256) {   // odd last extent: the staging phase without vector ALU work
    if (dtype == TGRAD_C64) TGRAD_LPF(TGRAD_C64); else TGRAD_LPF(TGRAD_CBF16);
  } else if (fuse) {                            // the host only fuses with W == 4 and one column tile
    if (dtype == TGRAD_C64) {
      if (K & 1) TGRAD_LP_FUSED(TGRAD_C64, true); else TGRAD_LP_FUSED(TGRAD_C64, false);
    } else {
      if (K & 1) TGRAD_LP_FUSED(TGRAD_CBF16, true); else TGRAD_LP_FUSED(TGRAD_CBF16, false);
    }
  } else if (dtype == TGRAD_C64) {
    if (ntb == 2) TGRAD_LP_W(TGRAD_C64, 2); else TGRAD_LP_W(TGRAD_C64, 1);
  } else {
    if (ntb == 2) TGRAD_LP_W(TGRAD_CBF16, 2); else TGRAD_LP_W(TGRAD_CBF16, 1);
  }
#undef TGRAD_LPF
#undef TGRAD_LPF_C
#undef TGRAD_LP_W
#undef TGRAD_LP_F
#undef TGRAD_LP_FUSED
#undef TGRAD_LP
#undef TGRAD_LP_C
}

void launch_lupdate(hipStream_t s, const float2* z, const float2* U, const Stage& st, int W, void* w,
                    int wdtype, float decay, float c_alpha, const int32_t* omega, const uint32_t* tile_start,
                    const float2* gs, float2* ms, float* vs, float beta1, float beta2, double inv_c1,
                    double inv_c2, float eps, float c_lambda) {
  const int64_t A = st.A;
  const int K = st.K, M = st.M;
  if (A * M <= 0) return;
  if (rows_update_pays(M, K, A))
    return launch_rows_update(s, z, U, st, w, wdtype, decay, c_alpha, omega, tile_start, gs, ms, vs, beta1, beta2, inv_c1,
                              inv_c2, eps, c_lambda);
  const int64_t ntiles = (A + kTileRows - 1) / kTileRows;
  const size_t lds = lupdate_lds_bytes(W, K, M);
  const int64_t ngroups = (ntiles + W - 1) / W;
  dim3 grid(1), block(64 * W);
  const SparseAdam sp = sparse_adam(omega, tile_start, gs, ms, vs, beta1, beta2, inv_c1, inv_c2, eps, c_lambda, 0);
  const float* zf = reinterpret_cast<const float*>(z);
  const int jt = lupdate_jt(K);
  const int up = (M + 3) / 4 <= 5 ? 5 : (M + 3) / 4 <= 9 ? 9 : kUpdPrefetch;
#define TGRAD_LU_U(W_, JT_, UP_)                                                                         \
  do {                                                                                                   \
    if (wdtype == TGRAD_C64) {                                                                           \
      allow_lds(k_lupdate<TGRAD_C64, W_, 2, JT_, UP_>, lds);   \
      grid.x = (unsigned)grid_for_tiles(ngroups, resident_blocks(k_lupdate<TGRAD_C64, W_, 2, JT_, UP_>, 64 * W_, lds));                                             \
      k_lupdate<TGRAD_C64, W_, 2, JT_, UP_><<<grid, block, lds, s>>>(zf, U, A, K, M, ntiles, w, decay, c_alpha, sp); \
    } else {                                                                                             \
      allow_lds(k_lupdate<TGRAD_CBF16, W_, 2, JT_, UP_>, lds);   \
      grid.x = (unsigned)grid_for_tiles(ngroups, resident_blocks(k_lupdate<TGRAD_CBF16, W_, 2, JT_, UP_>, 64 * W_, lds));                                           \
      k_lupdate<TGRAD_CBF16, W_, 2, JT_, UP_><<<grid, block, lds, s>>>(zf, U, A, K, M, ntiles, w, decay, c_alpha, sp); \
    }                                                                                                    \
  } while (0)
  // (narrow last modes of a rank above 8 are k_rows_update's: 4 wavefronts, variants of up to four operand pairs)
#define TGRAD_LU(W_, JT_)                                                                                \
  do {                                                                                                   \
    if constexpr (W_ == 4 && JT_ <= 4) {                                                                 \
      if (up == 5) { TGRAD_LU_U(4, JT_, 5); break; }                                                     \
      if (up == 9) { TGRAD_LU_U(4, JT_, 9); break; }                                                     \
    }                                                                                                    \
    TGRAD_LU_U(W_, JT_, kUpdPrefetch);                                                                   \
  } while (0)
#define TGRAD_LU_J(W_)                                                                                   \
  do {                                                                                                   \
    if (jt <= 1) TGRAD_LU(W_, 1); else if (jt == 2) TGRAD_LU(W_, 2); else if (jt == 4) TGRAD_LU(W_, 4);  \
    else if (jt == 8) TGRAD_LU(W_, 8); else TGRAD_LU(W_, 16);                                            \
  } while (0)
  if (W == 4) TGRAD_LU_J(4); else if (W == 2) TGRAD_LU_J(2); else TGRAD_LU_J(1);
#undef TGRAD_LU_U
#undef TGRAD_LU_J
#undef TGRAD_LU
}

// k_lupdate with the reconstruction stage of mode N-1 in front (see k_lupdate_fused): `y1` is the
// tensor before that stage, (slabs, K2, K) complex; `ut` the transposed factor copy; I2 = 32 S.
void launch_lupdate_fused(hipStream_t s, const float2* y1, const float2* ut, int I2, int K2, const float2* U,
                          const Stage& st, void* w, int wdtype, float decay, float c_alpha, const int32_t* omega,
                          const uint32_t* tile_start, int64_t k, const float2* gs, float2* ms, float* vs,
                          float beta1, float beta2, double inv_c1, double inv_c2, float eps, float c_lambda) {
  const int64_t A = st.A;
  const int K = st.K, M = st.M;
  if (A * M <= 0) return;
  constexpr int W = 4;
  const int64_t ntiles = A / kTileRows;
  const int S = I2 / kTileRows;
  const int64_t nslabs = ntiles / S;
  const int NT = (2 * M + 31) / 32;
  const size_t lds = (size_t)W * ((kTileRows * 2 * M + 3) & ~3) * 4 + (size_t)16 * 16 * NT * 8;
  const int64_t ngroups = (nslabs + W - 1) / W;
  dim3 grid(1), block(64 * W);
  const SparseAdam sp = sparse_adam(omega, tile_start, gs, ms, vs, beta1, beta2, inv_c1, inv_c2, eps, c_lambda,
                                    (int)(k > 0 ? k - 1 : 0));
  FusedPrev fz{y1, ut, S, K2};
  const int up = (M + 3) / 4 <= 5 ? 5 : (M + 3) / 4 <= 9 ? 9 : kUpdPrefetch;
  constexpr int kJT2 = 16;                     // (K2 in 17 .. 32: smaller ranks go to ends.hip)
#define TGRAD_LUF_M(UP_, MS_)                                                                            \
  do {                                                                                                   \
    if (wdtype == TGRAD_C64) {                                                                           \
      allow_lds(k_lupdate_fused<TGRAD_C64, W, MS_, kJT2, UP_>, lds);                                     \
      grid.x = (unsigned)grid_for_tiles(ngroups, resident_blocks(k_lupdate_fused<TGRAD_C64, W, MS_, kJT2, UP_>, 64 * W, lds)); \
      k_lupdate_fused<TGRAD_C64, W, MS_, kJT2, UP_><<<grid, block, lds, s>>>(U, A, K, M, ntiles, w, decay, c_alpha, sp, fz); \
    } else {                                                                                             \
      allow_lds(k_lupdate_fused<TGRAD_CBF16, W, MS_, kJT2, UP_>, lds);                                   \
      grid.x = (unsigned)grid_for_tiles(ngroups, resident_blocks(k_lupdate_fused<TGRAD_CBF16, W, MS_, kJT2, UP_>, 64 * W, lds)); \
      k_lupdate_fused<TGRAD_CBF16, W, MS_, kJT2, UP_><<<grid, block, lds, s>>>(U, A, K, M, ntiles, w, decay, c_alpha, sp, fz); \
    }                                                                                                    \
  } while (0)
  // the half-spectrum extents of FNO layers (2^m + 1) get a stage B with the extent as a compile-time constant
#define TGRAD_LUF(UP_, MS_)                                                                              \
  do {                                                                                                   \
    if (M == MS_) TGRAD_LUF_M(UP_, MS_); else TGRAD_LUF_M(UP_, 0);                                       \
  } while (0)
  if (up == 5) TGRAD_LUF(5, 17); else if (up == 9) TGRAD_LUF(9, 33); else TGRAD_LUF(kUpdPrefetch, 65);
#undef TGRAD_LUF
#undef TGRAD_LUF_M
}

}  // namespace tgrad
