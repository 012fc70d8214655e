// Mode-n products between the first compression stage and the last reconstruction stage, for a mode that
// is not the last: the tensor is (A, K, B) with B >= 1 contiguous columns.
//   k_mid      out[a, m, b] = sum_k F[m, k] x[a, k, b],  F = U^H (compression) or U
//   k_expand   the same for a short k (a rank): x stays in registers while the output rows go by
//   k_core     mode 1 both ways around AdamUpdate on the Tucker core, in one launch
// k_core, and the two others where a tensor fills the chip (k_mid_split, k_expand_split), run on split bf16 operands
// (device_common.h), k_mid and k_expand on float32 instructions.
// Tiles are 16 x 16 (v_mfma_f32_16x16x4f32, the same rate as 32x32x2).  Lanes g = lane / 16, c = lane % 16:
//   A[i = c][k = g] = F (row m = i),  B[k = g][j = c] = x (16 neighbouring columns: 128 or 256
//   contiguous bytes per row),  D register r: D[i = 4 g + r][j = c].
// re(F x) = Fr xr - Fi xi, im(F x) = Fr xi + Fi xr: four real products per step, column and tile.
// 16-wide tiles because ranks are padded to them (8 ... 24 in most layers: half the matrix work of 32-wide
// tiles) and because a wavefront then needs 16 columns instead of 32 or 64: twice to four times as many
// wavefronts in flight for the same tensor.  What bounds these stages is latency - a launch, one memory round
// trip for operands, one for x - until a tensor fills the chip, matrix work and memory in about equal parts after that.
// Measured (rocprofv3, us; 32x32x2 tiles with the factor always through LDS -> 16 x 16 in float32 -> as they are):
// 128x128x64x33, r 64,64,32,16: compressions + core + expansions 239 -> 147 -> 106; 128x128x128x65, r 32,32,32,16: 75 (16 x 16
// in float32) -> 55.
#include "device_common.h"
#include "launch_util.h"

namespace tgrad {

namespace {

template <int VEC> struct ColVec;
template <> struct ColVec<1> { typedef float2 type; };
template <> struct ColVec<2> { typedef float4 type; };

template <int VEC>
__device__ __forceinline__ void parts(const typename ColVec<VEC>::type& v, float* x) {   // (re, im) per column
  if constexpr (VEC == 1) {
    x[0] = v.x; x[1] = v.y;
  } else {
    x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
  }
}
// acc += f x for the VEC columns of x
template <int VEC>
__device__ __forceinline__ void cmac(v4f* acc, float2 f, const float* x) {
  const float nfy = -f.y;
#pragma unroll
  for (int i = 0; i < 2 * VEC; ++i) acc[i] = mfma16(f.x, x[i], acc[i]);
#pragma unroll
  for (int c = 0; c < VEC; ++c) {
    acc[2 * c] = mfma16(nfy, x[2 * c + 1], acc[2 * c]);
    acc[2 * c + 1] = mfma16(f.y, x[2 * c], acc[2 * c + 1]);
  }
}
template <int VEC>
__device__ __forceinline__ void store_cols(float* o, const v4f* acc, int r) {
  if constexpr (VEC == 1)
    *reinterpret_cast<float2*>(o) = make_float2(acc[0][r], acc[1][r]);
  else
    *reinterpret_cast<float4*>(o) = make_float4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
}
// F[m, k] of the stage, zero outside (M, K); U has rn columns
template <bool PROJECT>
__device__ __forceinline__ float2 factor_at(const FactorRef& U, int rn, int m, int k, int M, int K) {
  const float2 u = factor_entry(U, PROJECT ? k : m, PROJECT ? m : k, rn, m < M && k < K);
  return make_float2(u.x, PROJECT ? -u.y : u.y);
}

constexpr int kThreads = 256, kWaves = 4;
constexpr int kBatch = 8;                 // steps (4 rows each) of x per lane in flight
// Rows above which stages whose wavefronts have columns of their own take the split bf16 operands: below, a quad is mostly
// empty.  Both compressions of 100x100xKx60 behind the last, ranks 20 and r, float32 / split, us: K = 5, r 2 10.6 / 11.4; 6, 6
// 13.2 / 13.8; 8, 3 11.7 / 12.3; but 9, 4 13.5 / 12.5; 12, 5 15.4 / 14.2.
constexpr int kSplitRows = 8;
constexpr int kOwnSteps = kSplitRows / 4; // steps of those that do not

// The 16 column vectors of a wavefront: group `cg` of 16, lane column c; lanes past the end work on the
// last column and store nothing.
struct Cols {
  uint32_t cv, a, b;
  bool valid;
};
__device__ __forceinline__ Cols columns_of(uint32_t cg, int c, uint32_t ncv, uint32_t BV) {
  Cols q;
  const uint32_t raw = cg * 16u + (uint32_t)c;
  q.valid = raw < ncv;
  q.cv = q.valid ? raw : ncv - 1u;
  q.a = q.cv / BV;
  q.b = q.cv - q.a * BV;
  return q;
}

// SPLIT = false, at most kSplitRows rows: a wavefront owns 16 column vectors and MT tiles of 16 output rows (blockIdx.y:
//   which); the factor goes through LDS, shared by the 4 wavefronts.
// SPLIT = true, for few columns: the 4 wavefronts share 16 column vectors and split the rows k; each
//   fetches the operands of its own rows straight into registers (no LDS table, no barrier in front of the
//   matrix instructions) and the partial tiles meet in LDS, summed in a fixed order.
template <int VEC, int MT, bool PROJECT, bool SPLIT>
__global__ __launch_bounds__(kThreads) void k_mid(const float* __restrict__ x, const float2* __restrict__ Up, int rn,
                                                  uint32_t ncv, uint32_t BV, int K, int M, float* __restrict__ out) {
  typedef typename ColVec<VEC>::type V;
  extern __shared__ float2 sF[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const Cols cq = columns_of(SPLIT ? blockIdx.x : blockIdx.x * kWaves + wave, col, ncv, BV);
  const int64_t row = (int64_t)BV * VEC * 2;            // floats between consecutive k
  const float* xp = x + (int64_t)cq.a * K * row + (int64_t)cq.b * VEC * 2;
  const int mbase = blockIdx.y * (16 * MT);
  const int J = (K + 3) >> 2;
  // F[m, k] for k >= k0 = 4 j0 and the workgroup's rows: a full rank of an extent above 16384 does not fit one buffer
  auto factor_from = [&](int j0) -> FactorRef {
    const int64_t skip = PROJECT ? (int64_t)4 * j0 * rn : (int64_t)mbase * rn;
    return factor_ref(Up + skip, (int64_t)(PROJECT ? K : M) * rn - skip);
  };
  auto factor_in = [&](const FactorRef& U, int j0, int m, int k) -> float2 {
    const float2 u = factor_entry(U, PROJECT ? k - 4 * j0 : m - mbase, PROJECT ? m : k, rn, m < M && k < K);
    return make_float2(u.x, PROJECT ? -u.y : u.y);
  };
  auto load_x = [&](int j) -> V {                       // unconditional: rows past K meet zero factor entries
    const int k = 4 * j + grp;
    return *reinterpret_cast<const V*>(xp + (int64_t)(k < K ? k : K - 1) * row);
  };
  v4f acc[MT][2 * VEC];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int i = 0; i < 2 * VEC; ++i) acc[t][i] = (v4f){0.f, 0.f, 0.f, 0.f};

  if constexpr (SPLIT) {
    const int per = (J + kWaves - 1) / kWaves;
    const int j0 = wave * per, j1 = j0 + per < J ? j0 + per : J;
    for (int j = j0; j < j1; j += kBatch) {
      V v[kBatch];
      float2 f[kBatch][MT];
      const FactorRef U = factor_from(j);
#pragma unroll
      for (int u = 0; u < kBatch; ++u) v[u] = load_x(j + u);
#pragma unroll
      for (int u = 0; u < kBatch; ++u)                  // (steps past the slice: zero coefficients)
#pragma unroll
        for (int t = 0; t < MT; ++t)
          f[u][t] = factor_in(U, j, mbase + 16 * t + col, j + u < j1 ? 4 * (j + u) + grp : K);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        if (j + u < j1) {
          float xs[2 * VEC];
          parts<VEC>(v[u], xs);
#pragma unroll
          for (int t = 0; t < MT; ++t) cmac<VEC>(acc[t], f[u][t], xs);
        }
      }
    }
    // register r of every partial tile is summed (wavefronts in order) and stored by wavefront r
    float* red = reinterpret_cast<float*>(sF);          // [wave][tile][comp][r][lane]
    constexpr int kPart = MT * 2 * VEC * 4 * 64;
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int i = 0; i < 2 * VEC; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave * kPart + ((t * 2 * VEC + i) * 4 + r) * 64 + lane] = acc[t][i][r];
    __syncthreads();
    float* op = out + ((int64_t)cq.a * M) * row + (int64_t)cq.b * VEC * 2;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      float s[2 * VEC];
#pragma unroll
      for (int i = 0; i < 2 * VEC; ++i) {
        s[i] = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) s[i] += red[w * kPart + ((t * 2 * VEC + i) * 4 + wave) * 64 + lane];
      }
      const int m = mbase + 16 * t + 4 * grp + wave;
      if (cq.valid && m < M) {
        float* o = op + (int64_t)m * row;
        if constexpr (VEC == 1) *reinterpret_cast<float2*>(o) = make_float2(s[0], s[1]);
        else *reinterpret_cast<float4*>(o) = make_float4(s[0], s[1], s[2], s[3]);
      }
    }
  } else {
    V v[kOwnSteps];                                     // rows in flight before the factor is staged
#pragma unroll
    for (int j = 0; j < kOwnSteps; ++j) v[j] = load_x(j);
    const FactorRef U = factor_from(0);
    stage_table(sF, J * MT * 64, tid, kThreads, [&](int e) -> float2 {
      const int l = e & 63, t = (e >> 6) % MT, j = (e >> 6) / MT;
      return factor_in(U, 0, mbase + 16 * t + (l & 15), 4 * j + (l >> 4));
    });
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kOwnSteps; ++j) {
      if (j < J) {
        float xs[2 * VEC];
        parts<VEC>(v[j], xs);
#pragma unroll
        for (int t = 0; t < MT; ++t) cmac<VEC>(acc[t], sF[(j * MT + t) * 64 + lane], xs);
      }
    }
    if (!cq.valid) return;
    float* op = out + ((int64_t)cq.a * M) * row + (int64_t)cq.b * VEC * 2;
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = mbase + 16 * t + 4 * grp + r;
        if (m < M) store_cols<VEC>(op + (int64_t)m * row, acc[t], r);
      }
  }
}

// Reconstruction out[a, m, b] = sum_k U[m, k] x[a, k, b] with K <= 4 KS: a lane keeps its rows of x in
// registers (the B operands of every output tile) and the tiles of 16 output rows go by.
// SHARE = false: a wavefront owns 16 column vectors and the `tiles` tiles of blockIdx.y; operands from LDS.
// SHARE = true, for few columns: the 4 wavefronts share 16 column vectors and take one output tile each
//   (tile 4 blockIdx.y + wave), operands straight from memory: no barrier at all.
template <int VEC, int KS, bool SHARE>
__global__ __launch_bounds__(kThreads) void k_expand(const float* __restrict__ x, const float2* __restrict__ Up, int rn,
                                                     uint32_t ncv, uint32_t BV, int K, int M, int tiles,
                                                     float* __restrict__ out) {
  typedef typename ColVec<VEC>::type V;
  extern __shared__ float2 sF[];
  const FactorRef U = factor_ref(Up, (int64_t)M * rn);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const Cols cq = columns_of(SHARE ? blockIdx.x : blockIdx.x * kWaves + wave, col, ncv, BV);
  const int64_t row = (int64_t)BV * VEC * 2;
  const float* xp = x + (int64_t)cq.a * K * row + (int64_t)cq.b * VEC * 2;
  V v[KS];
#pragma unroll
  for (int j = 0; j < KS; ++j) {
    const int k = 4 * j + grp;
    v[j] = *reinterpret_cast<const V*>(xp + (int64_t)(k < K ? k : K - 1) * row);
  }
  float* op = out + ((int64_t)cq.a * M) * row + (int64_t)cq.b * VEC * 2;
  auto tile_out = [&](int q, auto operand) {
    v4f acc[2 * VEC];
#pragma unroll
    for (int i = 0; i < 2 * VEC; ++i) acc[i] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < KS; ++j) {
      float xs[2 * VEC];
      parts<VEC>(v[j], xs);
      cmac<VEC>(acc, operand(j), xs);
    }
    if (cq.valid) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * q + 4 * grp + r;
        if (m < M) store_cols<VEC>(op + (int64_t)m * row, acc, r);
      }
    }
  };
  if constexpr (SHARE) {
    const int q = blockIdx.y * kWaves + wave;
    if (16 * q >= M) return;
    float2 f[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j) f[j] = factor_at<false>(U, rn, 16 * q + col, 4 * j + grp, M, K);
    tile_out(q, [&](int j) { return f[j]; });
  } else {
    const int q0 = blockIdx.y * tiles, Q = (M + 15) >> 4;
    const int nq = Q - q0 < tiles ? Q - q0 : tiles;
    stage_table(sF, nq * KS * 64, tid, kThreads, [&](int e) -> float2 {
      const int l = e & 63, j = (e >> 6) % KS, q = (e >> 6) / KS;
      return factor_at<false>(U, rn, 16 * (q0 + q) + (l & 15), 4 * j + (l >> 4), M, K);
    });
    __syncthreads();
    for (int q = 0; q < nq; ++q) {
      const float2* ft = sF + q * KS * 64 + lane;
      tile_out(q0 + q, [&](int j) { return ft[j * 64]; });
    }
  }
}

// ---- the same two for tensors that fill the chip, on split bf16 operands ---------------------------
// In float32 matrix instructions these stages ran at half of those instructions' rate; in split operands (device_common.h) a
// product takes 96 cycles for 256.  128x128x64x33, r 64,64,32,16: compression 51 -> 28 us, expansion 56 -> 34, k_core 65 -> 48;
// 128x128x128x65, r 32,32,32,16: 27 -> 18, 29 -> 20, 20 -> 16.  Workgroups stay for several groups of columns, so that the
// factor is cut into its parts once for them (up to 96 KB of LDS).
// A quad is 16 rows k of the contraction: slot 2 j + part of lane (c, g) is part `part` of row 16 quad + 4 j + g.
// A operand: (Fr, Fi) of 16 output rows, from the table in LDS [quad][tile][h, m, l][lane]; B operands from one
// split of the column's (xr, xi): (xr, -xi) gives the real part of F x, (xi, xr) the imaginary part.
constexpr int kSplitItem = 3 * 64;        // u32v4 of one quad and tile of the table
constexpr int kChunkQuads = 8;            // quads staged at a time: 96 KB with four tiles

// table[(quad - q0) * tiles + tile] for quads q0 .. q0 + nq and output rows m0 .. m0 + 16 tiles
template <bool PROJECT>
__device__ __forceinline__ void stage_split(u32v4* table, const float2* Up, int rn, int M, int K, int m0, int tiles,
                                            int q0, int nq, int tid, int nthreads) {
  // (a full rank of an extent above 16384 does not fit one buffer: the buffer starts at the first row that is needed)
  const int64_t skip = PROJECT ? (int64_t)16 * q0 * rn : (int64_t)m0 * rn;
  const FactorRef U = factor_ref(Up + skip, (int64_t)(PROJECT ? K : M) * rn - skip);
  const int n = nq * tiles * 64;
  for (int e = tid; e < n; e += nthreads) {
    const int l = e & 63, it = e >> 6, t = it % tiles, q = it / tiles;
    const int m = 16 * t + (l & 15), k = 16 * q + (l >> 4);              // from m0 and 16 q0
    float2 f[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool in = m0 + m < M && 16 * q0 + k + 4 * j < K;
      f[j] = PROJECT ? factor_entry(U, k + 4 * j, m0 + m, rn, in) : factor_entry(U, m, 16 * q0 + k + 4 * j, rn, in);
      if (PROJECT) f[j].y = -f[j].y;
    }
    Split8 s;
#pragma unroll
    for (int j = 0; j < 4; ++j) split_at(s, j, f[j]);
    u32v4* d = table + it * kSplitItem + l;
    d[0] = s.h;
    d[64] = s.m;
    d[128] = s.l;
  }
}

// The same for an expansion's whole table, in two calls: the first BATCH items of a wavefront are requested before the columns
// of x are, so that what is needed first does not wait behind them (launch_mid has the line).  k_mid_split waits for its first
// rows of x alone beside the table, and the registers cost it more than the order gave (128x128x64x33, r 64,64,32,16: 31.9 ->
// 33 us).
template <int BATCH>
struct ExpandTable {
  FactorRef U;
  int rn, M, K, tiles, items;             // output rows and items of the table: tile + tiles * quad
  float2 f[BATCH][4];
  __device__ __forceinline__ ExpandTable(const float2* Up, int rn_, int M_, int K_, int m0, int tiles_, int quads)
      : U(factor_ref(Up + (int64_t)m0 * rn_, (int64_t)(M_ - m0) * rn_)), rn(rn_), M(M_ - m0), K(K_), tiles(tiles_),
        items(quads * tiles_) {}
  __device__ __forceinline__ void load(int it0, int waves, int l) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int it = it0 + u * waves, q = it / tiles, m = 16 * (it - q * tiles) + (l & 15), k = 16 * q + (l >> 4);
#pragma unroll
      for (int j = 0; j < 4; ++j) f[u][j] = factor_entry(U, m, k + 4 * j, rn, it < items && m < M && k + 4 * j < K);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ __forceinline__ void store(u32v4* table, int it0, int waves, int l) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int it = it0 + u * waves;
      if (it < items) {
        Split8 s;
#pragma unroll
        for (int j = 0; j < 4; ++j) split_at(s, j, f[u][j]);
        u32v4* d = table + it * kSplitItem + l;
        d[0] = s.h;
        d[64] = s.m;
        d[128] = s.l;
      }
    }
  }
  // everything, where `load(wave, ..)` has been called
  __device__ __forceinline__ void stage(u32v4* table, int wave, int waves, int l) {
    store(table, wave, waves, l);
    for (int it0 = wave + BATCH * waves; it0 < items; it0 += BATCH * waves) {
      load(it0, waves, l);
      store(table, it0, waves, l);
    }
  }
};
__device__ __forceinline__ Split8 split_item(const u32v4* p) { return Split8{p[0], p[64], p[128]}; }

// The operands of the VEC columns of four row vectors of a lane: [column][re, im]
template <int VEC>
__device__ __forceinline__ void split_rows(const typename ColVec<VEC>::type* v, Split8* b) {
  Split8 s[VEC];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float x[2 * VEC];
    parts<VEC>(v[j], x);
#pragma unroll
    for (int c = 0; c < VEC; ++c) split_at(s[c], j, make_float2(x[2 * c], x[2 * c + 1]));
  }
#pragma unroll
  for (int c = 0; c < VEC; ++c) {
    b[2 * c] = conj_pairs(s[c]);
    b[2 * c + 1] = swap_pairs(s[c]);
  }
}

template <int VEC, int MT, bool PROJECT, int W>
__global__ __launch_bounds__(64 * W) void k_mid_split(const float* __restrict__ x, const float2* __restrict__ Up, int rn,
                                                      uint32_t ncv, uint32_t BV, int K, int M, int groups,
                                                      float* __restrict__ out) {
  typedef typename ColVec<VEC>::type V;
  extern __shared__ u32v4 sQ[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const int64_t row = (int64_t)BV * VEC * 2;
  const int m0 = blockIdx.y * (16 * MT), Q = (K + 15) >> 4;
  const bool whole = Q <= kChunkQuads;                  // the table holds the whole factor
  for (int g0 = (int)blockIdx.x * W; g0 < groups; g0 += (int)gridDim.x * W) {   // (the same trips for every wavefront)
    const Cols cq = columns_of((uint32_t)(g0 + wave), col, ncv, BV);
    const float* xp = x + (int64_t)cq.a * K * row + (int64_t)cq.b * VEC * 2;
    auto load_x = [&](int k) -> V { return *reinterpret_cast<const V*>(xp + (int64_t)(k < K ? k : K - 1) * row); };
    V nxt[4];
    auto fetch = [&](int q) {                           // rows past K meet zero factor entries
#pragma unroll
      for (int j = 0; j < 4; ++j) nxt[j] = load_x(16 * q + 4 * j + grp);
    };
    fetch(0);
    v4f acc[MT][2 * VEC];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int i = 0; i < 2 * VEC; ++i) acc[t][i] = (v4f){0.f, 0.f, 0.f, 0.f};
    for (int q0 = 0; q0 < Q; q0 += kChunkQuads) {
      const int nq = Q - q0 < kChunkQuads ? Q - q0 : kChunkQuads;
      if (!whole || g0 == (int)blockIdx.x * W) {
        __syncthreads();                                // the chunk before is consumed
        stage_split<PROJECT>(sQ, Up, rn, M, K, m0, MT, q0, nq, tid, 64 * W);
        __syncthreads();
      }
      for (int q = 0; q < nq; ++q) {
        Split8 b[2 * VEC];
        split_rows<VEC>(nxt, b);
        fetch(q0 + q + 1);
        __builtin_amdgcn_sched_barrier(0);              // the loads stay in front of the quad they overlap
        const u32v4* ft = sQ + q * MT * kSplitItem + lane;
#pragma unroll
        for (int t = 0; t < MT; ++t) mfma_split<2 * VEC>(acc[t], split_item(ft + t * kSplitItem), b);
      }
    }
    if (cq.valid) {
      float* op = out + ((int64_t)cq.a * M) * row + (int64_t)cq.b * VEC * 2;
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + 16 * t + 4 * grp + r;
          if (m < M) store_cols<VEC>(op + (int64_t)m * row, acc[t], r);
        }
    }
  }
}

// Expansion of up to 16 KQ rows: their operands stay in registers while the tiles of 16 output rows go by.  AHEAD: items of the
// table that a wavefront requests before its columns (0: all of them after).
template <int VEC, int KQ, int W, int AHEAD>
__global__ __launch_bounds__(64 * W) void k_expand_split(const float* __restrict__ x, const float2* __restrict__ Up,
                                                         int rn, uint32_t ncv, uint32_t BV, int K, int M, int tiles,
                                                         int groups, float* __restrict__ out) {
  typedef typename ColVec<VEC>::type V;
  extern __shared__ u32v4 sQ[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const int64_t row = (int64_t)BV * VEC * 2;
  const int t0 = blockIdx.y * tiles, T = (M + 15) >> 4, nt = T - t0 < tiles ? T - t0 : tiles;
  const int stride = (int)gridDim.x * W;
  V v[KQ][4];
  Cols nq = columns_of((uint32_t)((int)blockIdx.x * W + wave), col, ncv, BV);
  auto fetch = [&](const Cols& c) {
    const float* xp = x + (int64_t)c.a * K * row + (int64_t)c.b * VEC * 2;
#pragma unroll
    for (int q = 0; q < KQ; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = 16 * q + 4 * j + grp;
        v[q][j] = *reinterpret_cast<const V*>(xp + (int64_t)(k < K ? k : K - 1) * row);
      }
  };
  if constexpr (AHEAD > 0) {
    ExpandTable<AHEAD> tab(Up, rn, M, K, 16 * t0, nt, KQ);
    tab.load(wave, W, lane);
    fetch(nq);
    tab.stage(sQ, wave, W, lane);
  } else {
    fetch(nq);
    stage_split<false>(sQ, Up, rn, M, K, 16 * t0, nt, 0, KQ, tid, 64 * W);
  }
  __syncthreads();
  for (int g = (int)blockIdx.x * W + wave; g < groups; g += stride) {
    const Cols cq = nq;
    Split8 b[KQ][2 * VEC];
#pragma unroll
    for (int q = 0; q < KQ; ++q) split_rows<VEC>(v[q], b[q]);
    if (g + stride < groups) {                          // the next columns go in flight
      nq = columns_of((uint32_t)(g + stride), col, ncv, BV);
      fetch(nq);
    }
    float* op = out + ((int64_t)cq.a * M) * row + (int64_t)cq.b * VEC * 2;
    for (int t = 0; t < nt; ++t) {
      v4f acc[2 * VEC];
#pragma unroll
      for (int i = 0; i < 2 * VEC; ++i) acc[i] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < KQ; ++q) mfma_split<2 * VEC>(acc, split_item(sQ + (q * nt + t) * kSplitItem + lane), b[q]);
      if (cq.valid) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = 16 * (t0 + t) + 4 * grp + r;
          if (m < M) store_cols<VEC>(op + (int64_t)m * row, acc, r);
        }
      }
    }
  }
}

// -------------------------------------------------------------------------------------------
// k_core: the three steps around the Tucker core in one kernel, for mode 1 (the slowest index):
//   g_L[m, b] = sum_k conj(U[k, m]) x[k, b]            last compression stage (K = I_1, M = r_1)
//   N_L = AdamUpdate(g_L)                               appendix algorithm "Adam with low-rank tensor
//                                                       decomposition" (moments updated in place)
//   z[i, b]   = sum_m U[i, m] N_L[m, b]                 first reconstruction stage
// so the core gradient and the core update never travel through memory between kernels (g_L is
// still written out: it is part of the readable state).
// A workgroup of W = 8 wavefronts owns 16 columns (4 where the extent fits them, up to 64 rows: half of the partial tiles, so
// twice the workgroups per compute unit; 23 rows, rank 17, 340000 columns 211 us with 8, 141 with 4; 16 rows, rank 16, 65536
// columns 24 and 17, 30 columns 3.7 and 3.0; launch_core has the lines).  Wavefront w contracts the steps of rows w, w + W, .. (4 rows
// each); the partial tiles are summed through LDS in a fixed order; AdamUpdate is spread over all threads
// and leaves N_L in LDS in accumulator layout, which IS the B operand layout of the expansion (register r
// of D holds rows 4 g + r: step r contracts exactly those); wavefront w then expands the output tiles
// w, w + W, ...  Every operand goes from memory straight into the registers of the one wavefront that
// uses it, and all of them (x, both factor operands, moments) are requested up front: one memory
// round trip, two barriers for a group of columns.
// Registers are what bounds it beside that: with indices in 64 bits the split operands made it 134 of them at one tile of
// rank, one workgroup per compute unit instead of two (16 rows, rank 16, 65536 columns 27 us in float32 instructions, then 32,
// now 17; 200 rows, rank 8, 20480 columns 22, then 26, now 20), and 176 bytes of scratch per lane at four (128 rows, rank 64,
// 48 columns 10.5, then 11, now 9.3; 65536 columns 102, then 82, now 72).
// A workgroup stays for several groups of columns where there are more of them than the chip holds: the factor operands
// are then fetched once per workgroup instead of once per 16 columns (ranks up to 64: 128 KB each, which the L2 caches
// delivered in 105 us for 128 x 32768 columns at rank 64, now 68), and a group's columns and moments arrive under the group before it.
// `z` may be `x` (in place): a workgroup writes only the columns it alone reads, a group's writes come after its reads
// (workgroup barriers in between), and what is fetched ahead are other columns.
struct CoreAdam {
  float2* m;            // first moments, (M, B) complex
  float* v;             // second moments
  float2* g_out;        // compressed gradient, written for the state accessors
  float beta1, beta2, inv_c1, inv_c2, eps;
};
constexpr int kCoreSteps = 4;             // steps of four rows of x per wavefront: one operand, all of them for K <= 16 waves

// MT: tiles of 16 that hold the rank; W: wavefronts of a workgroup
template <int MT, int W>
__global__ __launch_bounds__(64 * W) void k_core(const float* x, const float2* __restrict__ Up, int rn, int K,
                                                       int M, int64_t B, int groups, CoreAdam ad, float* z) {
  extern __shared__ float2 sF[];
  const FactorRef U = factor_ref(Up, (int64_t)K * rn);
  constexpr int kThr = 64 * W;
  constexpr int kPart = MT * 2 * 4 * 64;        // floats of one wavefront's partial tiles
  constexpr int kArea = W * kPart;     // [wave][tile][re / im][r][lane], then N_L as B operands [tile][h, m, l][lane]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const int64_t row = B * 2;
  const int J = (K + 3) >> 2, Q = (K + 15) >> 4;
  const bool once = J <= W * kCoreSteps;                       // (K <= 16 W) one batch of steps, one output tile each
  // operands of the compression: steps wave + W (s0 + u); past the end: zero coefficients
  float2 xv[kCoreSteps];
  Split8 fc[MT];
  // Eight wavefronts with four tiles of rank: the third parts of both sets of operands wait in LDS, a slot per lane
  // (registers for all parts there are not)
  constexpr bool kPark = MT == 4 && W == 8;
  u32v4* park = reinterpret_cast<u32v4*>(sF) + (kArea + MT * 768) / 4 + wave * (2 * MT * 64) + lane;
  auto set_low = [&](Split8* f, int set) {
    if constexpr (kPark) {
#pragma unroll
      for (int t = 0; t < MT; ++t) park[(set * MT + t) * 64] = f[t].l;
    }
  };
  auto operand = [&](const Split8* f, int set, int t) -> Split8 {
    return Split8{f[t].h, f[t].m, kPark ? park[(set * MT + t) * 64] : f[t].l};
  };
  auto fetch_x = [&](int g, int s0) {
    const uint32_t Bu = (uint32_t)B, b_raw = (uint32_t)g * 16u + (uint32_t)col, b = b_raw < Bu ? b_raw : Bu - 1u;
#pragma unroll
    for (int u = 0; u < kCoreSteps; ++u) {
      const int k = 4 * (wave + W * (s0 + u)) + grp;
      xv[u] = reinterpret_cast<const float2*>(x)[(uint32_t)(k < K ? k : K - 1) * Bu + b];   // (K B <= I < 2^31)
    }
  };
  auto fetch_in = [&](int s0) {
    float2 f[MT][kCoreSteps];
#pragma unroll
    for (int u = 0; u < kCoreSteps; ++u) {
      const int k = 4 * (wave + W * (s0 + u)) + grp;
#pragma unroll
      for (int t = 0; t < MT; ++t) f[t][u] = factor_at<true>(U, rn, 16 * t + col, k, M, K);
    }
    return [=](Split8* to) {
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int u = 0; u < kCoreSteps; ++u) split_at(to[t], u, f[t][u]);
      set_low(to, 0);
    };
  };
  // moments of this thread's core entries
  constexpr int kEnt = (MT * 256 + kThr - 1) / kThr;
  float2 mm[kEnt];
  float vv[kEnt];
  // (The first group's places in 64 bits: in 32 their products came in front of the other requests, 128 rows, rank 32, 256
  // groups 8.3 us, not 7.7.  The following ones' in 32: in 64 those of 1024 groups took 17.1 us, not 16.4.)
  auto entry = [&](int g, int q, auto wide, uint32_t& idx) -> bool {
    typedef decltype(wide) Int;
    const int e = tid + q * kThr;
    const int l = e & 63, r = (e >> 6) & 3, t = e >> 8;
    const int m = 16 * t + 4 * (l >> 4) + r;
    const Int bb = (Int)g * 16 + (Int)(l & 15);
    const bool live = t < MT && m < M && bb < (Int)B;
    idx = live ? (uint32_t)((Int)m * (Int)B + bb) : 0u;
    return live;
  };
  auto fetch_moments = [&](int g, auto wide) {
#pragma unroll
    for (int q = 0; q < kEnt; ++q) {
      uint32_t idx;
      entry(g, q, wide, idx);
      mm[q] = ad.m[idx];
      vv[q] = ad.v[idx];
    }
  };
  // operands of an output tile of the expansion
  Split8 fe[MT];
  auto fetch_out = [&](int q) {
    float2 f[MT][4];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) f[t][r] = factor_at<false>(U, rn, 16 * q + col, 16 * t + 4 * grp + r, K, M);
    return [=](Split8* to) {
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) split_at(to[t], r, f[t][r]);
      set_low(to, 1);
    };
  };
  int g = blockIdx.x;
  fetch_x(g, 0);
  {
    const auto in = fetch_in(0);
    fetch_moments(g, int64_t());
    if constexpr (MT == 4) {                                   // (both sets of operands at once do not fit the registers)
      in(fc);
      __builtin_amdgcn_sched_barrier(0);
      fetch_out(wave)(fe);
    } else {
      const auto out = fetch_out(wave);
      __builtin_amdgcn_sched_barrier(0);                       // (everything requested)
      in(fc);
      out(fe);
    }
  }
  float* red = reinterpret_cast<float*>(sF);
  uint32_t* sN = reinterpret_cast<uint32_t*>(red + kArea);
  for (int it = 0; g < groups; g += gridDim.x, ++it) {
    v4f acc[MT][2];
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t][0] = acc[t][1] = (v4f){0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0;; s0 += kCoreSteps) {
      Split8 b[2];
      split_rows<1>(xv, b);
#pragma unroll
      for (int t = 0; t < MT; ++t) mfma_split<2>(acc[t], operand(fc, 0, t), b);
      if (W * (s0 + kCoreSteps) >= J) break;          // (the same for every wavefront)
      fetch_x(g, s0 + kCoreSteps);
      fetch_in(s0 + kCoreSteps)(fc);
    }
    const int gn = g + gridDim.x;
    if (gn < groups) {                                         // the next group's columns go in flight
      fetch_x(gn, 0);
      if (!once) fetch_in(0)(fc);
    }
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave * kPart + ((t * 2 + i) * 4 + r) * 64 + lane] = acc[t][i][r];
    __syncthreads();
    // AdamUpdate; N_L goes to LDS as a B operand: row 16 t + 4 g + r is dword r of lane (c, g), tile t
#pragma unroll
    for (int q = 0; q < kEnt; ++q) {
      const int e = tid + q * kThr;
      const int l = e & 63, r = (e >> 6) & 3, t = e >> 8;
      if (MT * 256 % kThr == 0 || t < MT) {
        const float* pr = red + (t * 8 + r) * 64 + l;
        const float* pi = pr + 256;
        float gre = 0.f, gim = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) {
          gre += pr[w * kPart];
          gim += pi[w * kPart];
        }
        float2 m = mm[q];
        m.x = ad.beta1 * m.x + (1.f - ad.beta1) * gre;
        m.y = ad.beta1 * m.y + (1.f - ad.beta1) * gim;
        const float v = ad.beta2 * vv[q] + (1.f - ad.beta2) * (gre * gre + gim * gim);
        const float d = 1.f / (sqrtf(v * ad.inv_c2) + ad.eps);
        float nr = 0.f, ni = 0.f;
        uint32_t idx;
        if (entry(g, q, uint32_t(), idx)) {
          ad.m[idx] = m;
          ad.v[idx] = v;
          ad.g_out[idx] = make_float2(gre, gim);
          nr = m.x * ad.inv_c1 * d;
          ni = m.y * ad.inv_c1 * d;
        }
        uint32_t h, m3, l3;
        split_pair(nr, ni, h, m3, l3);
        uint32_t* pn = sN + (t * 192 + l) * 4 + r;
        pn[0] = h;
        pn[256] = m3;
        pn[512] = l3;
      }
    }
    if (gn < groups) fetch_moments(gn, uint32_t());
    __syncthreads();
    // expansion
    const int64_t b = (int64_t)g * 16 + col;
    float* op = z + b * 2;
    for (int q = wave; q < Q; q += W) {
      if (!once && (q != wave || it > 0)) fetch_out(q)(fe);
      v4f o[2];
      o[0] = o[1] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const Split8 n = split_item(reinterpret_cast<const u32v4*>(sN) + t * 192 + lane);
        const Split8 b2[2] = {conj_pairs(n), swap_pairs(n)};
        mfma_split<2>(o, operand(fe, 1, t), b2);
      }
      if (b < B) {
        const int i0 = 16 * q + 4 * grp;
        float* oi = op + (int64_t)i0 * row;
#pragma unroll
        for (int r = 0; r < 4; ++r, oi += row)
          if (i0 + r < K) store_cols<1>(oi, o, r);
      }
    }
  }
}

}  // namespace

// ---- host side ---------------------------------------------------------------------------------

// Column groups (16 column vectors each) from which on every wavefront takes one of its own (1024: one per SIMD);
// below, the wavefronts of a workgroup share a group so that the stage still spreads over the chip (372 groups,
// 90x77x66: 6.8 us shared, where 93 workgroups of one group per wavefront would leave 163 compute units idle).
constexpr int64_t kOwnColumns = 1024;

// k_expand's KS: steps of four rows of x, rounded up to the next variant.  Padded to 4, 8 or 16 steps a rank of a few was
// matrix work for nothing: 12M columns of one row 284 us, now 105; 3M from 2 rows to 4 78, now 34; 500000 from 20 to 24 43,
// now 36.
static int expand_steps(int K) {
  const int j = (K + 3) / 4;
  return j <= 6 ? j : j <= 8 ? 8 : j <= 10 ? 10 : j <= 12 ? 12 : 16;
}

void launch_mid(hipStream_t s, const float2* x, const float2* U, int rn, bool project, const Stage& st,
                float2* out) {
  const int64_t A = st.A, B = st.B;
  const int K = st.K, M = st.M;
  if (A * M * B <= 0) return;
  const float* xf = reinterpret_cast<const float*>(x);
  float* of = reinterpret_cast<float*>(out);
  // (two columns per lane, except where the operands of more than 32 rows would not stay in registers)
  const bool rows_fit = project || K <= 32 || K > 64;
  const int vec = rows_fit && B % 2 == 0 && A * (B / 2) / 16 >= kOwnColumns ? 2 : 1;
  const int64_t ncv64 = A * (B / vec);
  const uint32_t ncv = (uint32_t)ncv64, BV = (uint32_t)(B / vec);
  const int64_t groups = (ncv64 + 15) / 16;
  const bool own = groups >= kOwnColumns;
  const dim3 block(kThreads);
  const int Q = (M + 15) / 16;
  if (own && K > kSplitRows) {
    const int kq = (K + 15) / 16;
    if (!project && K <= 64) {
      // operands of `tiles` tiles: at most 96 KB
      const int most = 32 / kq, tiles = Q < most ? Q : most;
      const size_t lds = (size_t)tiles * kq * kSplitItem * 16;
      const unsigned ny = (unsigned)((Q + tiles - 1) / tiles);
      // The table's first items before the columns where a wavefront has three or more of them and the rows are more than one quad:
      // what it requests beyond its items only delays the columns.  A launch, us, columns first / four items of the table first (two of
      // more than two quads): 128x128x128x65, r 32,32,32,16 23.0 / 20.5; 128x128x32x33, r 20,32,16,16 15.7 / 15.2, with 128 of rank 64
      // 21.8 / 20.8; but with 64 of rank 16 10.3 / 10.7, 32 of rank 10 9.5 / 10.2, 64x32x32x33 with rank 10 6.7 / 7.2, 32 7.7 / 8.2, 64x64
      // with 32 10.4 / 11.1; with 200 of rank 32 (eight wavefronts) 25.8 / 25.8, two items first 25.2.
#define TGRAD_EXS(V_, KQ_, W_, AH_)                                                                  \
  do {                                                                                               \
    allow_lds(k_expand_split<V_, KQ_, W_, AH_>, lds);                                                \
    const int64_t most_ = (int64_t)compute_units() * resident_blocks(k_expand_split<V_, KQ_, W_, AH_>, 64 * W_, lds); \
    const int64_t need_ = (groups + W_ - 1) / W_;                                                    \
    k_expand_split<V_, KQ_, W_, AH_><<<dim3((unsigned)(need_ < most_ ? need_ : most_), ny), dim3(64 * W_), lds, s>>>( \
        xf, U, rn, ncv, BV, K, M, tiles, (int)groups, of);                                           \
  } while (0)
#define TGRAD_EXS_K(V_)                                                                              \
  do {                                                                                               \
    if (kq == 1) { if (lds > 48 * 1024) TGRAD_EXS(V_, 1, 8, 0); else TGRAD_EXS(V_, 1, 4, 0); }       \
    else if (lds > 48 * 1024) TGRAD_EXS(V_, 2, 8, 2);                                                \
    else if (tiles > 4) TGRAD_EXS(V_, 2, 4, 4);                                                      \
    else TGRAD_EXS(V_, 2, 4, 0);                                                                     \
  } while (0)
      if (kq == 3) { if (lds > 48 * 1024) TGRAD_EXS(1, 3, 8, 2); else TGRAD_EXS(1, 3, 4, 2); }
      else if (kq == 4) { if (lds > 48 * 1024) TGRAD_EXS(1, 4, 8, 2); else TGRAD_EXS(1, 4, 4, 2); }
      else if (vec == 2) TGRAD_EXS_K(2); else TGRAD_EXS_K(1);
#undef TGRAD_EXS_K
#undef TGRAD_EXS
      return;
    }
    const int mt = Q >= 4 ? 4 : Q >= 2 ? 2 : 1;
    const size_t lds = (size_t)(kq < kChunkQuads ? kq : kChunkQuads) * mt * kSplitItem * 16;
    const unsigned ny = (unsigned)((Q + mt - 1) / mt);
#define TGRAD_MIDS(V_, MT_, P_, W_)                                                                  \
  do {                                                                                               \
    allow_lds(k_mid_split<V_, MT_, P_, W_>, lds);                                                    \
    const int64_t most_ = (int64_t)compute_units() * resident_blocks(k_mid_split<V_, MT_, P_, W_>, 64 * W_, lds); \
    const int64_t need_ = (groups + W_ - 1) / W_;                                                    \
    k_mid_split<V_, MT_, P_, W_><<<dim3((unsigned)(need_ < most_ ? need_ : most_), ny), dim3(64 * W_), lds, s>>>( \
        xf, U, rn, ncv, BV, K, M, (int)groups, of);                                                  \
  } while (0)
#define TGRAD_MIDS_T(V_, P_)                                                                         \
  do {                                                                                               \
    if (mt == 4) TGRAD_MIDS(V_, 4, P_, 8); else if (mt == 2) TGRAD_MIDS(V_, 2, P_, 4); else TGRAD_MIDS(V_, 1, P_, 4); \
  } while (0)
    if (project) { if (vec == 2) TGRAD_MIDS_T(2, true); else TGRAD_MIDS_T(1, true); }
    else { if (vec == 2) TGRAD_MIDS_T(2, false); else TGRAD_MIDS_T(1, false); }
#undef TGRAD_MIDS_T
#undef TGRAD_MIDS
    return;
  }
  if (!project && K <= 64) {
    const int ks = expand_steps(K);
    const int tiles = own ? (Q < 64 / ks * 2 ? Q : 64 / ks * 2) : 1;          // operands of `tiles` tiles: at most 64 KB
    const size_t lds = own ? (size_t)tiles * ks * 512 : 0;
    const dim3 grid((unsigned)(own ? (groups + kWaves - 1) / kWaves : groups),
                    (unsigned)(own ? (Q + tiles - 1) / tiles : (Q + kWaves - 1) / kWaves));
#define TGRAD_EX(V_, KS_, S_)                                                                        \
  do {                                                                                               \
    allow_lds(k_expand<V_, KS_, S_>, lds);                                                           \
    k_expand<V_, KS_, S_><<<grid, block, lds, s>>>(xf, U, rn, ncv, BV, K, M, tiles, of);             \
  } while (0)
#define TGRAD_EX_K(V_, S_)                                                                           \
  do {                                                                                               \
    switch (ks) {                                                                                    \
      case 1: TGRAD_EX(V_, 1, S_); break;                                                            \
      case 2: TGRAD_EX(V_, 2, S_); break;                                                            \
      case 3: TGRAD_EX(V_, 3, S_); break;                                                            \
      case 4: TGRAD_EX(V_, 4, S_); break;                                                            \
      case 5: TGRAD_EX(V_, 5, S_); break;                                                            \
      case 6: TGRAD_EX(V_, 6, S_); break;                                                            \
      case 8: TGRAD_EX(V_, 8, S_); break;                                                            \
      case 10: TGRAD_EX(V_, 10, S_); break;                                                          \
      case 12: TGRAD_EX(V_, 12, S_); break;                                                          \
      default: TGRAD_EX(V_, 16, S_); break;                                                          \
    }                                                                                                \
  } while (0)
    // (with columns of their own the wavefronts have at most kSplitRows rows here: one or two steps)
    if (own && vec == 2) { if (ks == 1) TGRAD_EX(2, 1, false); else TGRAD_EX(2, 2, false); }
    else if (own) { if (ks == 1) TGRAD_EX(1, 1, false); else TGRAD_EX(1, 2, false); }
    else TGRAD_EX_K(1, true);
#undef TGRAD_EX_K
#undef TGRAD_EX
    return;
  }
  const int mt = Q >= 4 ? 4 : Q >= 2 ? 2 : 1;
  const dim3 grid((unsigned)(own ? (groups + kWaves - 1) / kWaves : groups), (unsigned)((Q + mt - 1) / mt));
  const size_t lds = own ? (size_t)((K + 3) / 4) * mt * 512 : (size_t)kWaves * mt * 2 * vec * 1024;
#define TGRAD_MID(V_, MT_, P_, S_)                                                                   \
  do {                                                                                               \
    allow_lds(k_mid<V_, MT_, P_, S_>, lds);                                                          \
    k_mid<V_, MT_, P_, S_><<<grid, block, lds, s>>>(xf, U, rn, ncv, BV, K, M, of);                   \
  } while (0)
#define TGRAD_MID_T(V_, P_, S_)                                                                      \
  do {                                                                                               \
    if (mt == 4) TGRAD_MID(V_, 4, P_, S_); else if (mt == 2) TGRAD_MID(V_, 2, P_, S_); else TGRAD_MID(V_, 1, P_, S_); \
  } while (0)
#define TGRAD_MID_P(V_, S_)                                                                          \
  do {                                                                                               \
    if (project) TGRAD_MID_T(V_, true, S_); else TGRAD_MID_T(V_, false, S_);                         \
  } while (0)
  // (with columns of their own the wavefronts have at most kSplitRows rows here, so no more than that of rank, and compress)
  if (own && vec == 2) TGRAD_MID(2, 1, true, false);
  else if (own) TGRAD_MID(1, 1, true, false);
  else TGRAD_MID_P(1, true);
#undef TGRAD_MID_P
#undef TGRAD_MID_T
#undef TGRAD_MID
}

// Where mode 1 (extent K, rank M) and the core's B columns are one launch.  Up to two tiles of rank it always is the better
// one.  Three or four tiles put one or two workgroups on a compute unit, and from some number of columns on the
// separate k_mid, k_adam_core and k_expand, which stream, are: the more matrix work per column, the later (they repeat
// none of it, but move the core twice more).  All stages but the first and the last, three kernels / one, us (modes 2 and 3
// not compressed beside it):
//   33 rows, rank 33: 20000 columns 70 / 66, 40960 85 / 88, 65536 108 / 119;    56, 44: 51200 109 / 107, 65536 120 / 120,
//   81920 159 / 162;    64, 64: 65536 132 / 126, 81920 171 / 170, 120832 236 / 252;
//   72, 52: 40960 110 / 105, 65536 151 / 152;    96, 33: 40960 116 / 114, 65536 152 / 157;
//   128, 64: 65536 197 / 185, 102400 339 / 345;  128, 33: 40960 136 / 130, 65536 178 / 182;
//   160, 33 (operands fetched per group): 10000 50 / 47;  200, 64: 12800 86 / 80, 20480 99 / 116;  250, 40: 16000 103 / 96.
bool core_kernel_fits(int K, int M, int64_t B) {
  if (M > 64 || K > TGRAD_MAX_EXTENT) return false;
  return M <= 32 || B <= (int64_t)K * M * (K <= 64 ? 24 : K <= 128 ? 14 : 2);
}

// Last compression stage + AdamUpdate on the core + first reconstruction stage (mode 1: the tensor
// before is (K, B), the tensor after is (K, B) again, the core in between (M, B)).
void launch_core(hipStream_t s, const float2* x, const float2* U, int rn, int K, int M, int64_t B, float2* m,
                 float* v, float2* g_out, float beta1, float beta2, float inv_c1, float inv_c2, float eps,
                 float2* z) {
  if (B <= 0) return;
  CoreAdam ad{m, v, g_out, beta1, beta2, inv_c1, inv_c2, eps};
  const float* xf = reinterpret_cast<const float*>(x);
  float* zf = reinterpret_cast<float*>(z);
  const int64_t groups = (B + 15) / 16;
#define TGRAD_CORE(MT_, W_)                                                                                  \
  do {                                                                                                       \
    const size_t lds = (size_t)W_ * MT_ * 2048 + (size_t)MT_ * 3072 + (MT_ == 4 && W_ == 8 ? W_ * MT_ * 2048 : 0); \
    allow_lds(k_core<MT_, W_>, lds);                                                                         \
    const int64_t cap = (int64_t)compute_units() * resident_blocks(k_core<MT_, W_>, 64 * W_, lds);           \
    k_core<MT_, W_><<<dim3((unsigned)(groups < cap ? groups : cap)), dim3(64 * W_), lds, s>>>(xf, U, rn, K, M, B, (int)groups, ad, zf); \
  } while (0)
  // (one tile of rank: four wavefronts as well where eight do not hold the rows either and there is more than a group per
  // compute unit, 140 rows, 32768 columns 32 us with 8, 28 with 4; but 128 rows 19.4 / 22.2, and 120 groups of 250 7.5 / 8.7)
  if (M <= 16 && (K <= 64 || (K > 128 && groups > compute_units()))) TGRAD_CORE(1, 4);
  else if (M <= 16) TGRAD_CORE(1, 8);
  else if (M <= 32 && K <= 64) TGRAD_CORE(2, 4);
  else if (M <= 32) TGRAD_CORE(2, 8);
  else if (K <= 64) TGRAD_CORE(4, 4);
  else TGRAD_CORE(4, 8);
#undef TGRAD_CORE
}

}  // namespace tgrad
