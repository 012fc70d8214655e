// Factor refresh: {U^(n)} <- TuckerFactors(R_L, r), third line of the refresh branch of
// Algorithm 1, as HOSVD (appendix "Implementation": truncated SVD of every mode-n unfolding).
// The left singular vectors of the unfolding R_L(n) are the eigenvectors of the Hermitian
// mode-n Gram matrix A_n = R_L(n) R_L(n)^H, so the refresh is
//   (1) A_n for every compressed mode, accumulated in float64 on the f64 matrix cores, with
//       R_L = G - Sparse(G, Omega) formed on load from the support bitmask, and
//   (2) an eigen-solve of each A_n in float64 for its r_n leading eigenvectors, written
//       eigenvalue-descending with the phase of every column fixed (largest-modulus entry real and
//       positive): for extents up to 128 tridiagonalisation (one workgroup per mode), then one
//       wavefront per eigenvector for multisection, inverse iteration and back-transformation; cyclic
//       Jacobi for clustered spectra and larger extents.
// float64 is used because Adam in core space is not invariant to the basis inside the subspace:
// noise-like gradients have relative eigenvalue gaps near 1e-4, and float32 accumulation error
// divided by such a gap would move the individual eigenvectors far more than the update tolerates.
#include <type_traits>

#include "device_common.h"
#include "launch_util.h"

namespace tgrad {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kSuper = 128;          // rows of the output handled by one workgroup, per side
constexpr int kTC = 16;              // tensor columns staged per tile
constexpr int kRowD = 4 * kTC + 2;   // doubles per staged row: 4 per element + a pad of 16 bytes (conflict-free reads)
constexpr int kGramThreads = 1024;   // 16 wavefronts: a 4 x 4 grid of 32 x 32 output blocks

// Gram of the tensor viewed as (A, In, B): gram[i, j] = sum_{a, b} x[a, i, b] conj(x[a, j, b]).
// Real embedding on v_mfma_f64_16x16x4f64 (K = 4 = two tensor columns x {re, im}):
//   Re[i, j] = sum xr_i xr_j + xi_i xi_j      -> A operand (xr_i | xi_i),  B operand (xr_j | xi_j)
//   Im[i, j] = sum xi_i xr_j - xr_i xi_j      -> A operand (xi_i | -xr_i), B operand (xr_j | xi_j)
// Operand lanes: A[i = lane % 16][k = lane / 16], B[k = lane / 16][j = lane % 16];
// result: register r of lane l holds D[4 r + l / 16][l % 16].
// The matrix is Hermitian, so only its lower triangle is computed: a workgroup owns one 128 x 128
// super block (si >= sj) of one chunk of tensor columns, cut into 16 x 16 matrix-core tiles - all 64
// of them off the diagonal, the 36 on or below it on the diagonal - dealt round-robin to its 16
// wavefronts (tile t to wavefront t % 16: 9 tiles per SIMD in the diagonal case).  The next
// 16 columns are fetched into registers while the current ones are in the matrix cores.
// A staged element is converted to float64 once, when it is committed to LDS, and stored as the four
// operands it can be asked for: (xr, xi, xi, -xr).  The f64 matrix instructions run on the SIMD's
// vector ALU; a conversion and a select per operand fetch in the inner loop (each element is an
// operand of up to 8 tiles) took as many of its cycles as the matrix instructions themselves.
constexpr int kGramMaxTiles = 4;     // tiles per wavefront: 64 / 16

template <int DT>
__global__ __launch_bounds__(kGramThreads) void k_gram(const void* __restrict__ x,
                                                        const uint32_t* __restrict__ mask, int64_t A,
                                                        int In, int64_t B, int64_t cols_per_chunk,
                                                        double* __restrict__ partials) {
  extern __shared__ double sG[];
  double* sI = sG;                                    // [row][column][xr, xi, xi, -xr]
  double* sJ = sG + kSuper * kRowD;
  const int nsup = (In + kSuper - 1) / kSuper;
  const int si = blockIdx.y / nsup, sj = blockIdx.y % nsup;
  if (si < sj) return;                                // upper super blocks: mirrored by the reduction
  const bool diag = si == sj;
  const int64_t J = A * B;
  const int64_t c_begin = (int64_t)blockIdx.x * cols_per_chunk;
  const int64_t c_end = c_begin + cols_per_chunk < J ? c_begin + cols_per_chunk : J;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part = (lane >> 4) & 1;
  const int ccol = lane >> 5;
  const int lrow = lane & 15;
  const int rows_i = In - si * kSuper < kSuper ? In - si * kSuper : kSuper;   // rows present in the two
  const int rows_j = In - sj * kSuper < kSuper ? In - sj * kSuper : kSuper;   // super blocks

  // this wavefront's tiles: slot k holds tile t = wave + 16 k (static slots: no dynamic indexing)
  int ti[kGramMaxTiles], tj[kGramMaxTiles];
  bool mine[kGramMaxTiles];
  const int ntl = diag ? 36 : 64;
#pragma unroll
  for (int k = 0; k < kGramMaxTiles; ++k) {
    const int t = wave + 16 * k;
    int a = 0, b = 0;
    if (diag) {
      a = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
      while (a * (a + 1) / 2 > t) --a;
      while ((a + 1) * (a + 2) / 2 <= t) ++a;
      b = t - a * (a + 1) / 2;
    } else {
      a = t >> 3;
      b = t & 7;
    }
    mine[k] = t < ntl && 16 * a < rows_i && 16 * b < rows_j;   // tiles of absent rows hold zeros: skipped
    ti[k] = mine[k] ? a : 0;
    tj[k] = mine[k] ? b : 0;
  }

  v4d accRe[kGramMaxTiles], accIm[kGramMaxTiles];
#pragma unroll
  for (int k = 0; k < kGramMaxTiles; ++k) {
    accRe[k] = (v4d){0., 0., 0., 0.};
    accIm[k] = (v4d){0., 0., 0., 0.};
  }

  // A thread stages elements e = tid + u * 1024 (u < kPer) of a tile: row il, column cl.  Which ones
  // they are does not depend on the tile, so everything that can be is computed once: the LDS slot,
  // the tensor offset of (row, cl) inside a tile, and whether the row exists.
  constexpr int kPer = kSuper * kTC / kGramThreads;   // 2 elements per thread and side
  int e_cl[kPer], e_lds[kPer];
  int64_t e_offI[kPer], e_offJ[kPer];                 // (row * B + cl) for the row side / the column side
  bool e_okI[kPer], e_okJ[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int e = tid + u * kGramThreads;
    int il, cl;
    if (B == 1) {                                     // rows are the fastest index in memory
      il = e % kSuper;
      cl = e / kSuper;
    } else {                                          // columns b are the fastest index
      il = e / kTC;
      cl = e % kTC;
    }
    e_cl[u] = cl;
    e_lds[u] = il * kRowD + 4 * cl;
    e_okI[u] = si * kSuper + il < In;
    e_okJ[u] = sj * kSuper + il < In;
    e_offI[u] = (int64_t)(si * kSuper + il) * B + cl;
    e_offJ[u] = (int64_t)(sj * kSuper + il) * B + cl;
  }
  // Column c = c0 + cl of the unfolding is tensor index (a, b) = (c / B, c % B); with (a0, b0) those
  // of the tile's first column (kept up to date by the caller) the element (row i, column c) lies at
  //   (a0 In + i) B + b0 + cl            if b0 + cl < B,
  //   ... + (In - 1) B                   if the column has wrapped into the next a (at most once
  //                                      per tile when B >= 16; smaller B take the general form).
  // A 64-bit division per fetched element would cost the vector ALU - which the f64 matrix
  // instructions also run on - more cycles than the tile's matrix instructions.
  const int64_t wrap_add = (int64_t)(In - 1) * B;
  auto fetch = [&](bool row_ok, int64_t off, int cl, int64_t c0, int64_t a0, int64_t b0) -> float2 {
    float2 v = make_float2(0.f, 0.f);
    if (row_ok && c0 + cl < c_end) {
      int64_t idx;
      if (B >= kTC) {
        idx = a0 * In * B + b0 + off + (b0 + cl >= B ? wrap_add : (int64_t)0);
      } else {                                        // tiny trailing extent: b0 + cl < 32
        const uint32_t q = (uint32_t)(b0 + cl) / (uint32_t)B;
        idx = a0 * In * B + b0 + off + (int64_t)q * wrap_add;
      }
      // both loads are issued together (a load that waits for the mask bit would double the latency)
      const uint32_t mw = mask ? mask[idx >> 5] : 0u;
      const float2 xv = load_elem<DT>(x, idx);
      if (!((mw >> (idx & 31)) & 1u)) v = xv;
    }
    return v;
  };

  float2 preI[kPer], preJ[kPer];                      // next tile of the row side / the column side
  int64_t pa0 = c_begin / B, pb0 = c_begin - pa0 * B; // of the tile being fetched (workgroup-uniform)
  auto next_tile = [&]() {                            // (a0, b0) of the tile kTC columns further on
    pb0 += kTC;
    if (B >= kTC) {
      if (pb0 >= B) { pb0 -= B; pa0 += 1; }
    } else {
      const uint32_t q = (uint32_t)pb0 / (uint32_t)B;
      pa0 += q;
      pb0 -= (int64_t)q * B;
    }
  };
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    preI[u] = fetch(e_okI[u], e_offI[u], e_cl[u], c_begin, pa0, pb0);
    preJ[u] = diag ? make_float2(0.f, 0.f) : fetch(e_okJ[u], e_offJ[u], e_cl[u], c_begin, pa0, pb0);
  }

  // pre -> one staged tile (row side into dI; column side into dJ when the super block is off the diagonal)
  auto commit = [&](double* dI, double* dJ) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      {
        const double xr = (double)preI[u].x, xi = (double)preI[u].y;
        double2* d = reinterpret_cast<double2*>(dI + e_lds[u]);
        d[0] = make_double2(xr, xi);
        d[1] = make_double2(xi, -xr);
      }
      if (!diag) {
        const double xr = (double)preJ[u].x, xi = (double)preJ[u].y;
        *reinterpret_cast<double2*>(dJ + e_lds[u]) = make_double2(xr, xi);
      }
    }
  };
  auto prefetch = [&](int64_t c0) {                   // the tile that starts at column c0 -> pre
    next_tile();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      preI[u] = fetch(e_okI[u], e_offI[u], e_cl[u], c0, pa0, pb0);
      if (!diag) preJ[u] = fetch(e_okJ[u], e_offJ[u], e_cl[u], c0, pa0, pb0);
    }
  };
  // Operand addresses are invariant lane offsets plus constants: a wavefront takes its tiles one after
  // the other and, per tile, the 8 column pairs of the staged tile unrolled, so that nothing in the
  // loop but the matrix instructions needs the vector ALU (which they occupy).
  int offA[kGramMaxTiles], offB[kGramMaxTiles];       // doubles, from the start of a staged area
#pragma unroll
  for (int k = 0; k < kGramMaxTiles; ++k) {
    offA[k] = (16 * ti[k] + lrow) * kRowD + 4 * ccol + part;
    offB[k] = (16 * tj[k] + lrow) * kRowD + 4 * ccol + part;
  }
  auto multiply = [&](const double* bI, const double* bJ) {
#pragma unroll
    for (int k = 0; k < kGramMaxTiles; ++k) {
      if (mine[k]) {
        const double* pa = bI + offA[k];
        const double* pb = bJ + offB[k];
#pragma unroll
        for (int s2 = 0; s2 < kTC / 2; ++s2) {        // column 2 s2 + ccol: 4 doubles per column
          const double aRe = pa[8 * s2];              // part ? xi : xr
          const double aIm = pa[8 * s2 + 2];          // part ? -xr : xi
          const double bop = pb[8 * s2];
          accRe[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(aRe, bop, accRe[k], 0, 0, 0);
          accIm[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(aIm, bop, accIm[k], 0, 0, 0);
        }
      }
    }
  };
  if (diag) {
    // One staged side only, so the two LDS areas take turns: while the wavefronts multiply tile t out
    // of one, tile t + 1 is committed into the other (it was read last for tile t - 1, before the
    // barrier that ended that tile) and tile t + 2 is fetched into registers.  One barrier per tile.
    commit(sI, sI);
    if (c_begin + kTC < c_end) prefetch(c_begin + kTC);
    __syncthreads();
    int it = 0;
    for (int64_t c0 = c_begin; c0 < c_end; c0 += kTC, ++it) {
      double* cur = (it & 1) ? sJ : sI;
      double* nxt = (it & 1) ? sI : sJ;
      if (c0 + kTC < c_end) commit(nxt, nxt);
      if (c0 + 2 * kTC < c_end) prefetch(c0 + 2 * kTC);
      multiply(cur, cur);
      __syncthreads();
    }
  } else {
    for (int64_t c0 = c_begin; c0 < c_end; c0 += kTC) {
      __syncthreads();                                // previous tile fully consumed
      commit(sI, sJ);
      __syncthreads();
      if (c0 + kTC < c_end) prefetch(c0 + kTC);       // next 16 columns go in flight
      multiply(sI, sJ);
    }
  }
  double2* out = reinterpret_cast<double2*>(partials) + (int64_t)blockIdx.x * In * In;
#pragma unroll
  for (int k = 0; k < kGramMaxTiles; ++k) {
    if (mine[k]) {
      for (int r = 0; r < 4; ++r) {
        const int i = si * kSuper + 16 * ti[k] + 4 * r + (lane >> 4);
        const int j = sj * kSuper + 16 * tj[k] + (lane & 15);
        if (i < In && j < In) out[(int64_t)i * In + j] = make_double2(accRe[k][r], accIm[k][r]);
      }
    }
  }
}

// -------------------------------------------------------------------------------------------------
// k_gram128: the Gram for extents In <= 128 (every mode of the FNO shapes), all modes of a tensor in one launch.
// A complex Hermitian product in THREE real ones.  With P1 = Xr Xr^T, P2 = Xi Xi^T and P3 = (Xr + Xi)(Xr - Xi)^T,
//   Re = P1 + P2,   Im = Xi Xr^T - Xr Xi^T = P3 - P1 + P2,
// so a 16 x 16 tile takes three matrix instructions per four tensor columns instead of four.  The products of
// float32 numbers are exact in float64 and so, up to 29 bits of difference in exponent, are the sums Xr +- Xi.  The
// rounding of Im is bounded by the row norms' product like that of the four-product form, with the constant of three
// sums in place of two.  Measured against 80-bit sums, in units of 2^-53 times the row norms' product, root mean square
// (before / now): 128 rows of 4200 columns Re 0.59 / 0.36, Im 0.03 / 0.03; 16 rows of 120000 Re 3.9 / 0.62, Im 0.01 / 0.01
// (columns are split more ways now).
// What runs next to the f64 matrix instructions matters, because they occupy the SIMD's vector ALU:
//  * RT tile rows (1, 2, 4 or 8) are held; a staged tile is 4096 elements whatever RT: 256 / RT columns, so a thread
//    always has 8 loads in flight and a barrier is passed as rarely as the LDS allows.
//  * LDS holds two planes (re, im) per staged tile, column by column, rows contiguous, an odd column stride.  (Not free of
//    bank conflicts: 1.13 cycles of them for every one of active LDS instructions; operands are requested three column
//    pairs ahead.)  Xr +- Xi are formed in registers.
//  * Fetch: the element and its support-mask word come through buffer descriptors (the tile's first column as
//    base, scalar); lanes without an element use an offset that the range check answers with zero.
//    The mask is applied at the commit, so nothing waits for the loads before the matrix phase.
//  * RT = 8: the 36 tiles of the lower triangle over 8 wavefronts, runs inside one tile row (fewer than 8 tile rows
//    present: dealt one by one).  RT <= 4: the wavefronts also split the columns of the staged tile - 10 tiles = 2 x 5,
//    columns 4 ways; 3 or 1 tiles, columns 8 ways - and add their parts through LDS at the end: every SIMD has the
//    same number of matrix instructions.
//  * An extent of 16 RT + 1 (a half-spectrum mode) has its last row done by vector arithmetic, lane = column row:
//    65 rows would need 15 tiles instead of 10.
// Measured (rocprofv3, us per mode of 128x128x128x65; before: four products, 16-column tiles, 15 tiles for 65 rows):
// 128 rows 1330 - 1385 -> 1010 (the matrix instructions alone: 765), 65 rows 1510 -> 707; a refresh 6558 -> 4809.
struct GramRuns {                    // a wavefront's tiles when all 8 tile rows exist: run A = (ra, a0 .. a0 + na - 1),
  signed char ra, a0, na, rb, b0, nb;  // run B = (rb, b0 .. b0 + nb - 1), every run inside one tile row
};
// 36 tiles of the lower triangle over 8 wavefronts: 5 tiles for wavefronts 0..3, 4 tiles for 4..7
// (wavefronts w and w + 4 share a SIMD: 9 tiles per SIMD).  Wavefronts 5..7 hold one run of 4.
__constant__ GramRuns kGramRuns[8] = {
    {2, 0, 3, 1, 0, 2}, {4, 0, 3, 3, 0, 2}, {5, 0, 3, 3, 2, 2}, {5, 3, 3, 4, 3, 2},
    {6, 0, 3, 0, 0, 1}, {6, 3, 2, 6, 5, 2}, {7, 0, 2, 7, 2, 2}, {7, 4, 2, 7, 6, 2}};

constexpr int kGram128Threads = 512;

struct GramJob {
  int rt;                            // tile rows held: the variant of the kernel
  const void* x;
  const uint32_t* mask;
  double* partials;
  int64_t A, B;
  int In;
  uint32_t magicB;
  uint32_t start, weight, tiles;     // where its tiles lie on the line of all work, and how long each is
};
struct GramJobs {
  uint32_t per, rem;                 // workgroup b has the line from gram_edge(b) to gram_edge(b + 1)
  int njobs;
  int first[kMaxNdim], nchunks[kMaxNdim];   // workgroups first .. first + nchunks - 1 have a part of a job
  GramJob job[kMaxNdim];
};
__host__ __device__ inline uint32_t gram_edge(uint32_t per, uint32_t rem, uint32_t b) { return b * per + (b < rem ? b : rem); }
// tiles of a job that start before `at`
__host__ __device__ inline uint32_t gram_tiles_before(uint32_t at, uint32_t start, uint32_t weight, uint32_t tiles) {
  if (at <= start) return 0u;
  const uint32_t t = (at - start + weight - 1) / weight;
  return t < tiles ? t : tiles;
}

__host__ __device__ constexpr int gram_cols(int RT) { return 256 / RT; }            // tensor columns per staged tile
__host__ __device__ constexpr int gram_plane(int RT) { return gram_cols(RT) * (16 * RT + 1); }   // doubles

__device__ __forceinline__ __amdgpu_buffer_rsrc_t gram_buffer(const void* base, uint32_t bytes) {
  // untyped buffer, stride 0: a load at an offset >= bytes returns zero
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// tile t of the lower triangle of a tile grid
__device__ constexpr int tri_row(int t) { int a = 0; while ((a + 1) * (a + 2) / 2 <= t) ++a; return a; }

template <int DT, int RT>
__device__ __forceinline__ void gram_chunk(const GramJob& jb, uint32_t tile0, uint32_t tile1, int chunk, double* sG) {
  constexpr int TC = gram_cols(RT), Q = 16 * RT + 1, PL = gram_plane(RT);
  constexpr int kEs = DT == TGRAD_C64 ? 8 : 4;        // bytes per element
  constexpr uint32_t kNowhere = 0xFFFFFFF0u;          // an offset beyond every descriptor: the load returns zero
  constexpr int kTiles = RT == 8 ? 6 : RT == 4 ? 5 : RT == 2 ? 3 : 1;    // per wavefront
  constexpr int CG = RT == 8 ? 1 : RT == 4 ? 4 : 8;   // wavefronts that share tiles and split the columns
  const int In = jb.In;
  const int64_t J = jb.A * jb.B;
  const uint32_t B = (uint32_t)jb.B;                  // the host takes this kernel only when In * B < 2^28
  const int64_t c_begin = (int64_t)tile0 * TC;
  const int64_t c_end = (int64_t)tile1 * TC < J ? (int64_t)tile1 * TC : J;
  const bool empty = c_begin >= c_end;                // (workgroup-uniform) a chunk without columns writes zeros
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 15, lcol = lane >> 4;
  const int ntr = (In + 15) >> 4;                     // tile rows present
  const bool tail = RT < 8 && In == 16 * RT + 1;

  // ---- staging: thread's elements (il, cl) = first + u * step, u < 8; the ninth is the tail row's ----
  constexpr int kPer = 4096 / kGram128Threads;
  const bool last = B == 1;                           // the mode is the fastest index in memory: lanes along rows
  const int il0 = last ? tid % (16 * RT) : tid / TC, cl0 = last ? tid / (16 * RT) : tid % TC;
  const int ilstep = last ? 0 : kGram128Threads / TC, clstep = last ? 32 / RT : 0;
  const uint32_t ustep = last ? (uint32_t)clstep * (uint32_t)In : (uint32_t)ilstep * B;   // elements between them
  const int slot0 = cl0 * Q + il0, slotstep = clstep * Q + ilstep;
  const uint32_t wrap_add = (uint32_t)(In - 1) * B;   // a column past B continues one leading index further
  const uint64_t total_bytes = (uint64_t)J * (uint64_t)In * kEs;
  const __amdgpu_buffer_rsrc_t rmask =
      gram_buffer(jb.mask, jb.mask ? (uint32_t)((((uint64_t)J * In + 31) >> 5) * 4) : 0u);
  uint32_t pa0 = (uint32_t)(c_begin / jb.B), pb0 = (uint32_t)(c_begin - (int64_t)pa0 * jb.B);   // tile being fetched
  uint32_t pre0[kPer + 1], pre1[kPer + 1], pre_m[kPer + 1], pre_g[kPer + 1];
  auto wraps = [&](uint32_t c) -> uint32_t {          // (b0 + column) / B
    const uint32_t nn = pb0 + c;
    return B >= (uint32_t)TC ? (nn >= B ? 1u : 0u) : jb.magicB ? __umulhi(nn, jb.magicB) : nn;
  };
  auto fetch_tile = [&](int64_t c0) {                 // the tile that starts at column c0 = (pa0, pb0) -> pre
    const uint64_t base_e = (uint64_t)pa0 * (uint64_t)In * B + pb0;      // < 2^31 elements
    const uint64_t left = total_bytes - base_e * kEs;
    const __amdgpu_buffer_rsrc_t rx = gram_buffer(reinterpret_cast<const char*>(jb.x) + base_e * kEs,
                                                  left > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)left);
    const int lim = (int)(c_end - c0 < TC ? c_end - c0 : TC);            // columns of this tile inside the chunk
    auto load = [&](int u, bool ok, uint32_t off) {
      const uint32_t gi = (uint32_t)base_e + off;
      pre_g[u] = gi;
      const uint32_t voff = ok ? off * kEs : kNowhere;
      if constexpr (DT == TGRAD_C64) {
        typedef uint32_t u2 __attribute__((ext_vector_type(2)));
        const u2 rr = __builtin_amdgcn_raw_buffer_load_b64(rx, voff, 0, 0);
        pre0[u] = rr.x;
        pre1[u] = rr.y;
      } else {
        pre0[u] = __builtin_amdgcn_raw_buffer_load_b32(rx, voff, 0, 0);
        pre1[u] = 0u;
      }
      pre_m[u] = __builtin_amdgcn_raw_buffer_load_b32(rmask, ok ? ((gi >> 5) << 2) : kNowhere, 0, 0);
    };
    const uint32_t first = last ? (uint32_t)(il0 + cl0 * In) : (uint32_t)il0 * B + (uint32_t)cl0 + wraps((uint32_t)cl0) * wrap_add;
#pragma unroll
    for (int u = 0; u < kPer; ++u)
      load(u, il0 + u * ilstep < In && il0 + u * ilstep < 16 * RT && cl0 + u * clstep < lim, first + (uint32_t)u * ustep);
    if (tail)
      load(kPer, tid < lim, last ? (uint32_t)(tid * In + In - 1)
                                 : (uint32_t)(In - 1) * B + (uint32_t)tid + wraps((uint32_t)tid) * wrap_add);
  };
  auto next_tile = [&]() {
    pb0 += TC;
    if (B >= (uint32_t)TC) {
      if (pb0 >= B) { pb0 -= B; pa0 += 1; }
    } else {
      const uint32_t q = jb.magicB ? __umulhi(pb0, jb.magicB) : pb0;
      pa0 += q;
      pb0 -= q * B;
    }
  };
  auto commit = [&](double* d) {                      // pre -> one staged tile: plane of re, plane of im
    auto put = [&](int u, int slot) {
      // all ones where the entry is in the support: one instruction (a shift, a test and two selects were five, in a loop whose
      // vector instructions stand between the matrix ones)
      const uint32_t gone = (uint32_t)__builtin_amdgcn_sbfe((int)pre_m[u], pre_g[u], 1);
      const uint32_t w0 = pre0[u] & ~gone, w1 = pre1[u] & ~gone;
      float fr, fi;
      if constexpr (DT == TGRAD_C64) {
        fr = __uint_as_float(w0);
        fi = __uint_as_float(w1);
      } else {                                        // a bf16 is the upper half of a float32
        fr = __uint_as_float(w0 << 16);
        fi = __uint_as_float(w0 & 0xFFFF0000u);
      }
      d[slot] = (double)fr;
      d[PL + slot] = (double)fi;
    };
#pragma unroll
    for (int u = 0; u < kPer; ++u) put(u, slot0 + u * slotstep);
    if (tail && tid < TC) put(kPer, tid * Q + 16 * RT);
  };

  v4d p1[kTiles], p2[kTiles], p3[kTiles];
#pragma unroll
  for (int k = 0; k < kTiles; ++k) p1[k] = p2[k] = p3[k] = (v4d){0., 0., 0., 0.};
  double t_re = 0., t_im = 0., t_dd = 0.;             // tail row against this lane's row, and itself
  int ti[kTiles], tj[kTiles];
  bool mine[kTiles];
  const int tg = RT == 4 ? wave >> 2 : 0, cg = RT == 8 ? 0 : RT == 4 ? wave & 3 : wave;
  if constexpr (RT == 8) {
    if (ntr == 8) {
      const GramRuns g = kGramRuns[wave];
#pragma unroll
      for (int k = 0; k < kTiles; ++k) {
        const bool in_a = k < g.na;
        mine[k] = k < g.na + g.nb;
        ti[k] = in_a ? g.ra : g.rb;
        tj[k] = !mine[k] ? 0 : in_a ? g.a0 + k : g.b0 + (k - g.na);
      }
    } else {                                          // fewer tile rows: tile t of the lower triangle to wavefront t % 8
      const int ntl = ntr * (ntr + 1) / 2;
#pragma unroll
      for (int k = 0; k < kTiles; ++k) {
        const int t = wave + 8 * k;
        int a = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
        while (a * (a + 1) / 2 > t) --a;
        while ((a + 1) * (a + 2) / 2 <= t) ++a;
        mine[k] = t < ntl;
        ti[k] = mine[k] ? a : 0;
        tj[k] = mine[k] ? t - a * (a + 1) / 2 : 0;
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < kTiles; ++k) {
      const int t = tg * kTiles + k, a = tri_row(t);
      ti[k] = a;
      tj[k] = t - a * (a + 1) / 2;
      mine[k] = a < ntr;
    }
  }
  const int lane_off = lcol * Q + lrow;
  auto three = [&](int k, double ar, double ai, double br, double bi) {
    p1[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, p1[k], 0, 0, 0);
    p2[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, bi, p2[k], 0, 0, 0);
    p3[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar + ai, br - bi, p3[k], 0, 0, 0);
  };
  // A run of NT tiles of one tile row in accumulator slots S0 ..: the row-side operands are fetched once per four
  // columns for the whole run, one step ahead of the matrix instructions.
  auto multiply_run = [&](const double* b, auto s0_c, auto nt_c) {
    constexpr int S0 = decltype(s0_c)::value, NT = decltype(nt_c)::value, STEPS = TC / 4;
    const double* pa = b + 16 * ti[S0] + lane_off;
    const double* pb[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) pb[k] = b + 16 * tj[S0 + k] + lane_off;
    double ar[2], ai[2], br[2][NT], bi[2][NT];
    auto fetch_ops = [&](int s) {
      const int slot = s & 1;
      ar[slot] = pa[4 * s * Q];
      ai[slot] = pa[4 * s * Q + PL];
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        br[slot][k] = pb[k][4 * s * Q];
        bi[slot][k] = pb[k][4 * s * Q + PL];
      }
    };
    fetch_ops(0);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (s + 1 < STEPS) fetch_ops(s + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < NT; ++k) three(S0 + k, ar[s & 1], ai[s & 1], br[s & 1][k], bi[s & 1][k]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto multiply_single = [&](const double* b) {       // tile by tile
#pragma unroll
    for (int k = 0; k < kTiles; ++k) {
      if (mine[k]) {
        const double* pa = b + 16 * ti[k] + lane_off;
        const double* pb = b + 16 * tj[k] + lane_off;
#pragma unroll
        for (int s = 0; s < TC / 4; ++s) three(k, pa[4 * s * Q], pa[4 * s * Q + PL], pb[4 * s * Q], pb[4 * s * Q + PL]);
      }
    }
  };
  // RT <= 4: all tiles of group G on this wavefront's steps; every tile row's operands are read once per step
  auto multiply_group = [&](const double* b, auto g_c) {
    constexpr int G = decltype(g_c)::value, STEPS = TC / 4 / CG;
    constexpr int NR = RT == 4 ? (G == 0 ? 3 : 4) : RT;                  // tile rows the group touches
    const double* pa = b + cg * 4 * Q + lane_off;
    double xr[2][NR], xi[2][NR];
    auto fetch_ops = [&](int s) {
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        xr[s & 1][q] = pa[4 * CG * s * Q + 16 * q];
        xi[s & 1][q] = pa[4 * CG * s * Q + 16 * q + PL];
      }
    };
    fetch_ops(0);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (s + 1 < STEPS) fetch_ops(s + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < kTiles; ++k) {
        constexpr int t0 = G * kTiles;
        const int a = tri_row(t0 + k), c = t0 + k - a * (a + 1) / 2;     // (constants after unrolling)
        if (a < ntr) three(k, xr[s & 1][a], xi[s & 1][a], xr[s & 1][c], xi[s & 1][c]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // row 16 RT against every row: lane groups of 16 RT rows take a column each
  constexpr int LG = RT >= 4 ? 1 : 4 / RT;
  auto tail_row = [&](const double* b) {
    const int jl = lane % (16 * RT < 64 ? 16 * RT : 64), lg = LG > 1 ? lane / (16 * RT) : 0;
#pragma unroll
    for (int c = 0; c < TC / (8 * LG); ++c) {
      const double* col = b + (LG * (wave + 8 * c) + lg) * Q;
      const double yr = col[16 * RT], yi = col[16 * RT + PL], xr = col[jl], xi = col[jl + PL];
      t_re += yr * xr + yi * xi;
      t_im += yi * xr - yr * xi;
      t_dd += yr * yr + yi * yi;
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  using I4 = std::integral_constant<int, 4>;

  // ---- main loop: while the wavefronts multiply tile t out of one LDS area, tile t + 1 is committed into the other
  // (read last for tile t - 1, before the barrier that ended it) and tile t + 2 is fetched.  One instance of the loop
  // per shape of a wavefront's tile set; every instance passes the same barriers. ----
  auto main_loop = [&](auto multiply) {
    double* buf0 = sG;
    double* buf1 = sG + 2 * PL;
    fetch_tile(c_begin);
    commit(buf0);
    if (c_begin + TC < c_end) { next_tile(); fetch_tile(c_begin + TC); }
    __syncthreads();
    int it = 0;
    for (int64_t c0 = c_begin; c0 < c_end; c0 += TC, ++it) {
      double* cur = (it & 1) ? buf1 : buf0;
      double* nxt = (it & 1) ? buf0 : buf1;
      if (c0 + TC < c_end) commit(nxt);
      if (c0 + 2 * TC < c_end) { next_tile(); fetch_tile(c0 + 2 * TC); }
      multiply(cur);
      if (tail) tail_row(cur);
      __syncthreads();
    }
  };
  if (!empty) {
    if constexpr (RT == 8) {
      if (ntr != 8) main_loop([&](const double* b) { multiply_single(b); });
      else if (wave < 4) main_loop([&](const double* b) { multiply_run(b, I0{}, I3{}); multiply_run(b, I3{}, I2{}); });
      else if (wave == 4) main_loop([&](const double* b) { multiply_run(b, I0{}, I3{}); multiply_run(b, I3{}, I1{}); });
      else main_loop([&](const double* b) { multiply_run(b, I0{}, I4{}); });   // both runs lie in one tile row: a run of 4
    } else if constexpr (RT == 4) {
      if (tg == 0) main_loop([&](const double* b) { multiply_group(b, I0{}); });
      else main_loop([&](const double* b) { multiply_group(b, I1{}); });
    } else {
      main_loop([&](const double* b) { multiply_group(b, I0{}); });
    }
  }
  // Re = P1 + P2 and Im = P3 - P1 + P2 replace p1 and p2
#pragma unroll
  for (int k = 0; k < kTiles; ++k) {
    const v4d re = p1[k] + p2[k];
    p2[k] = p3[k] - p1[k] + p2[k];
    p1[k] = re;
  }
  if constexpr (CG > 1) {
    // the column groups' parts: upper half onto the lower one until one is left (RT = 4: one group at a time, they do
    // not fit in pairs), always the same order
    constexpr int kPart = kTiles * 8 * 64;
    int hi = CG;
#pragma unroll
    for (int round = 0; round < 3; ++round) {
      const int half = RT == 4 ? hi - 1 : hi / 2;
      double* area = sG + (tg * (RT == 4 ? 1 : CG / 2) + (cg >= half ? cg - half : cg)) * kPart + lane;
      if (cg >= half && cg < hi) {
#pragma unroll
        for (int k = 0; k < kTiles; ++k)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            area[(k * 8 + r) * 64] = p1[k][r];
            area[(k * 8 + 4 + r) * 64] = p2[k][r];
          }
      }
      __syncthreads();
      if (cg < hi - half) {
#pragma unroll
        for (int k = 0; k < kTiles; ++k)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            p1[k][r] += area[(k * 8 + r) * 64];
            p2[k][r] += area[(k * 8 + 4 + r) * 64];
          }
      }
      __syncthreads();
      hi = half;
    }
  }
  double2* out = reinterpret_cast<double2*>(jb.partials) + (int64_t)chunk * In * In;
  if (cg == 0) {
#pragma unroll
    for (int k = 0; k < kTiles; ++k) {
      if (mine[k]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = 16 * ti[k] + 4 * r + (lane >> 4);
          const int j = 16 * tj[k] + (lane & 15);
          if (i < In && j < In && i < 16 * RT) out[(int64_t)i * In + j] = make_double2(p1[k][r], p2[k][r]);
        }
      }
    }
  }
  if (tail) {                                         // the wavefronts' columns of the tail row, in order
    double* area = sG + lane;
    area[(wave * 3) * 64] = t_re;
    area[(wave * 3 + 1) * 64] = t_im;
    area[(wave * 3 + 2) * 64] = t_dd;
    __syncthreads();
    if (wave == 0) {
      double re = 0., im = 0., dd = 0.;
#pragma unroll
      for (int w = 0; w < 8; ++w)
#pragma unroll
        for (int g = 0; g < LG; ++g) {               // (lanes past the rows read on, and write nothing)
          const int at = LG > 1 ? (lane % (16 * RT)) + g * 16 * RT - lane : 0;
          re += area[(w * 3) * 64 + at];
          im += area[(w * 3 + 1) * 64 + at];
          dd += area[(w * 3 + 2) * 64 + at];
        }
      if (lane < 16 * RT) out[(int64_t)(16 * RT) * In + lane] = make_double2(re, im);
      if (lane == 0) out[(int64_t)(16 * RT) * In + 16 * RT] = make_double2(dd, 0.);
    }
  }
}

template <int DT>
__global__ __launch_bounds__(kGram128Threads) void k_gram128(GramJobs jobs) {
  extern __shared__ double sG[];
  const uint32_t at0 = gram_edge(jobs.per, jobs.rem, blockIdx.x), at1 = gram_edge(jobs.per, jobs.rem, blockIdx.x + 1);
  uint32_t todo = 0u;
#pragma unroll
  for (int j = 0; j < kMaxNdim; ++j)
    todo |= j < jobs.njobs && (uint32_t)((int)blockIdx.x - jobs.first[j]) < (uint32_t)jobs.nchunks[j] ? 1u << j : 0u;
  for (; todo; todo &= todo - 1u) {
    const int j = __builtin_ctz(todo);
    const GramJob jb = jobs.job[j];
    const int chunk = (int)blockIdx.x - jobs.first[j];
    const uint32_t t0 = gram_tiles_before(at0, jb.start, jb.weight, jb.tiles);
    const uint32_t t1 = gram_tiles_before(at1, jb.start, jb.weight, jb.tiles);
    __syncthreads();                                  // (the LDS of the part of the job before)
    if (jb.rt == 8) gram_chunk<DT, 8>(jb, t0, t1, chunk, sG);
    else if (jb.rt == 4) gram_chunk<DT, 4>(jb, t0, t1, chunk, sG);
    else if (jb.rt == 2) gram_chunk<DT, 2>(jb, t0, t1, chunk, sG);
    else gram_chunk<DT, 1>(jb, t0, t1, chunk, sG);
  }
}

// gram[i, j] = sum over chunks of partials[chunk][i, j] for i >= j; the upper triangle is the
// conjugate mirror (the Gram kernels leave it unwritten).  The chunks of one entry are summed by 8
// threads, each over a contiguous eighth of the chunks in order, and the 8 partial sums are added in
// order: the result does not depend on the launch, and 8 times as many loads are in flight.
constexpr int kReduceSplit = 8;
constexpr int kReduceElems = 256 / kReduceSplit;     // entries per workgroup
struct ReduceJobs {
  const double* partials[kMaxNdim];
  double* gram[kMaxNdim];
  int In[kMaxNdim], nchunks[kMaxNdim];
};
__global__ __launch_bounds__(256) void k_gram_reduce(ReduceJobs jobs) {
  __shared__ double2 part[kReduceSplit][kReduceElems];
  const int In = jobs.In[blockIdx.y], nchunks = jobs.nchunks[blockIdx.y];
  const int el = threadIdx.x % kReduceElems, sub = threadIdx.x / kReduceElems;
  const int64_t e = (int64_t)blockIdx.x * kReduceElems + el;
  const int64_t n2 = (int64_t)In * In;
  if ((int64_t)blockIdx.x * kReduceElems >= n2) return;
  const bool in = e < n2;
  const int i = in ? (int)(e / In) : 0, j = in ? (int)(e - (int64_t)i * In) : 0;
  const int64_t src = i >= j ? (int64_t)i * In + j : (int64_t)j * In + i;
  const int per = (nchunks + kReduceSplit - 1) / kReduceSplit;
  const int c0 = sub * per, c1 = c0 + per < nchunks ? c0 + per : nchunks;
  const double2* p2 = reinterpret_cast<const double2*>(jobs.partials[blockIdx.y]);
  double re = 0., im = 0.;
  if (in) {
#pragma unroll 8
    for (int c = c0; c < c1; ++c) {
      const double2 v = p2[(int64_t)c * n2 + src];
      re += v.x;
      im += v.y;
    }
  }
  part[sub][el] = make_double2(re, im);
  __syncthreads();
  if (sub == 0 && in) {
    double sr = 0., si = 0.;
#pragma unroll
    for (int q = 0; q < kReduceSplit; ++q) {
      sr += part[q][el].x;
      si += part[q][el].y;
    }
    reinterpret_cast<double2*>(jobs.gram[blockIdx.y])[e] = make_double2(sr, i > j ? si : i < j ? -si : 0.);
  }
}

// ---------------------------------------------------------------------------------------------
// Hermitian eigen-solve by parallel cyclic Jacobi (two-sided rotations, round-robin pairing).
// One workgroup per matrix; A and V live in global memory (L2-resident, <= 1 MiB each).
struct EigJob {
  const double* gram;   // n x n complex (interleaved), row-major
  double* A;            // work copy
  double* V;            // eigenvector accumulator
  float* U;             // out: n x r complex float32, row-major
  int* status;          // out: [0] = 1 if the solve stopped at the sweep limit with rotations left, else 0;
                        //      [1] = Jacobi sweeps run; [2] = 1 if the tridiagonal path declined (close eigenvalues)
  int n;
  int r;
  int max_sweeps;
  int use_fast;         // 1: Householder tridiagonalisation + bisection + inverse iteration first (n <= 128), the
                        //    Jacobi kernels run only if that path declines (status[2] != 0); 0: Jacobi
};
struct EigJobs {
  EigJob job[kMaxNdim];
};

// Rotation log of the LDS solver (extents <= 128), kept in the job's work buffer `A`: a header,
// then one entry per (logged round, slot).  p < 0: the slot's pivot was already negligible.
struct RotLog {
  double c, sx, sy;     // cos, sin e^{i phi}
  int p, q;
};
struct EigLogHeader {
  double lam[128];      // eigenvalues (diagonal of the converged work matrix)
  int rounds;           // logged rounds (rounds in which nothing rotates are not logged)
  int pad[3];
};

constexpr int kEigThreads = 1024;
constexpr int kEigMaxN = TGRAD_MAX_EXTENT;
constexpr int kEigMaxSweeps = 30;
constexpr int kEigBatch = 4;           // rotations per thread whose loads are in flight together

__device__ __forceinline__ double2 cmuld(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 conjd(double2 a) { return make_double2(a.x, -a.y); }

// Shared tail of the eigensolvers: order the eigenvalues in `lam` descending (ties: lower index
// first), keep the first r, give every kept column of V the unit phase that makes its
// largest-modulus entry (first on ties) real and positive, and write U (n x r, float32).
__device__ void eig_finish(int n, int r, int tid, const double* lam, int* col_of, double2* phase,
                           const double2* V, float2* U) {
  for (int i = tid; i < n; i += kEigThreads) {
    int rank = 0;
    const double li = lam[i];
    for (int j = 0; j < n; ++j) rank += (lam[j] > li || (lam[j] == li && j < i)) ? 1 : 0;
    if (rank < r) col_of[rank] = i;
  }
  __syncthreads();
  for (int cidx = tid; cidx < r; cidx += kEigThreads) {
    const int src = col_of[cidx];
    double best = -1.;
    double2 vb = make_double2(1., 0.);
    for (int i = 0; i < n; ++i) {
      const double2 v = V[i * n + src];
      const double a2 = v.x * v.x + v.y * v.y;
      if (a2 > best) {
        best = a2;
        vb = v;
      }
    }
    const double mag = sqrt(best);
    phase[cidx] = mag > 0. ? make_double2(vb.x / mag, -vb.y / mag) : make_double2(1., 0.);
  }
  __syncthreads();
  for (int e = tid; e < n * r; e += kEigThreads) {
    const int i = e / r, cidx = e - i * r;
    const double2 v = cmuld(V[i * n + col_of[cidx]], phase[cidx]);
    U[e] = make_float2((float)v.x, (float)v.y);
  }
}

// Pair (p, q), p < q, of round `round` for slot `slot` of the round-robin tournament on m players.
__device__ __forceinline__ void jacobi_pair(int slot, int round, int m, int& p, int& q) {
  if (slot == 0) {
    p = m - 1;
    q = round;
  } else {
    p = (round + slot) % (m - 1);
    q = (round - slot + (m - 1)) % (m - 1);
  }
  if (p > q) {
    const int t = p;
    p = q;
    q = t;
  }
}

// Rotation that annihilates a_pq of the Hermitian 2 x 2 pivot [[app, apq], [conj(apq), aqq]]:
// c = cos, s = sin e^{i phi}.  Returns false (c = 1, s = 0) when a_pq is already negligible.
__device__ __forceinline__ bool jacobi_rotation(double app, double aqq, double2 apq, double eps2, double floor2,
                                                double& c, double2& s) {
  c = 1.;
  s = make_double2(0., 0.);
  const double mag2 = apq.x * apq.x + apq.y * apq.y;
  if (!(mag2 > eps2 * fabs(app * aqq) && mag2 > floor2)) return false;
  // two reciprocal square roots, one square root and one division (the threads that compute the
  // rotations are the critical path of a round: every other wavefront waits for them)
  const double inv_mag = rsqrt(mag2);
  const double tau = 0.5 * (aqq - app) * inv_mag;
  const double t = (tau >= 0. ? 1. : -1.) / (fabs(tau) + sqrt(1. + tau * tau));
  c = rsqrt(1. + t * t);
  const double sn = t * c * inv_mag;
  s = make_double2(sn * apq.x, sn * apq.y);
  return true;
}

__global__ __launch_bounds__(kEigThreads) void k_eig(EigJobs jobs) {
  const EigJob jb = jobs.job[blockIdx.x];
  const int n = jb.n, r = jb.r;
  const int tid = threadIdx.x;
  double2* A = reinterpret_cast<double2*>(jb.A);
  double2* V = reinterpret_cast<double2*>(jb.V);
  const double2* G = reinterpret_cast<const double2*>(jb.gram);

  __shared__ int sp[kEigMaxN / 2 + 1], sq[kEigMaxN / 2 + 1];
  __shared__ double sc[kEigMaxN / 2 + 1];       // cos
  __shared__ double2 ss[kEigMaxN / 2 + 1];      // sin * e^{i phi}
  __shared__ int srot[kEigMaxN / 2 + 1];        // 1 if this pair rotates in this round
  __shared__ int nrot;
  __shared__ double red[kEigThreads];
  __shared__ double lam[kEigMaxN];
  __shared__ int col_of[kEigMaxN];
  __shared__ double2 phase[kEigMaxN];

  // A <- gram, V <- I, trace
  double tr = 0.;
  for (int e = tid; e < n * n; e += kEigThreads) {
    double2 g = G[e];
    A[e] = g;
    const int i = e / n, j = e - i * n;
    V[e] = make_double2(i == j ? 1. : 0., 0.);
    if (i == j) tr += g.x;
  }
  red[tid] = tr;
  __syncthreads();
  for (int off = kEigThreads / 2; off > 0; off >>= 1) {
    if (tid < off) red[tid] += red[tid + off];
    __syncthreads();
  }
  const double trace = red[0];
  const double floor2 = (2.2e-18 * trace / n) * (2.2e-18 * trace / n);   // (1e-2 eps mean-eigenvalue)^2
  const double eps2 = 4.93e-32;                                          // (2^-52)^2
  const int m = n + (n & 1);                                             // even player count
  const int half = m / 2;

  int sweeps_run = 0, converged = 0;
  for (int sweep = 0; sweep < jb.max_sweeps; ++sweep) {
    if (tid == 0) nrot = 0;
    __syncthreads();
    for (int round = 0; round < m - 1; ++round) {
      // ---- phase 1: pairs of this round and their rotations ----
      if (tid < half) {
        int p, q;
        jacobi_pair(tid, round, m, p, q);
        int rot = 0;
        double c = 1.;
        double2 s = make_double2(0., 0.);
        if (q < n)                                     // q == n is the padding player of an odd n
          rot = jacobi_rotation(A[p * n + p].x, A[q * n + q].x, A[p * n + q], eps2, floor2, c, s) ? 1 : 0;
        sp[tid] = p;
        sq[tid] = q;
        sc[tid] = c;
        ss[tid] = s;
        srot[tid] = rot;
        if (rot) atomicAdd(&nrot, 1);
      }
      __syncthreads();
      // ---- phase 2: column rotations  X[:, p] <- c X[:, p] - conj(s) X[:, q],
      //                                 X[:, q] <- s X[:, p] + c X[:, q]   for X in {A, V} ----
      // (loads of a batch are all issued before the first use: one memory round trip per batch)
      for (int e0 = tid; e0 < 2 * n * half; e0 += kEigThreads * kEigBatch) {
        double2 xp[kEigBatch], xq[kEigBatch];
        int off_p[kEigBatch], off_q[kEigBatch], prs[kEigBatch];      // prs: pair | (matrix << 16), -1 = idle
#pragma unroll
        for (int u = 0; u < kEigBatch; ++u) {
          const int e = e0 + u * kEigThreads;
          prs[u] = -1;
          if (e < 2 * n * half) {
            const int which = e / (n * half);
            const int e2 = e - which * (n * half);
            const int i = e2 / half, pr = e2 - i * half;
            if (srot[pr]) {
              const double2* X = which ? V : A;
              prs[u] = pr | (which << 16);
              off_p[u] = i * n + sp[pr];
              off_q[u] = i * n + sq[pr];
              xp[u] = X[off_p[u]];
              xq[u] = X[off_q[u]];
            }
          }
        }
#pragma unroll
        for (int u = 0; u < kEigBatch; ++u) {
          if (prs[u] >= 0) {
            double2* X = (prs[u] >> 16) ? V : A;
            const int pr = prs[u] & 0xFFFF;
            const double c = sc[pr];
            const double2 s = ss[pr];
            const double2 t1 = cmuld(conjd(s), xq[u]), t2 = cmuld(s, xp[u]);
            X[off_p[u]] = make_double2(c * xp[u].x - t1.x, c * xp[u].y - t1.y);
            X[off_q[u]] = make_double2(t2.x + c * xq[u].x, t2.y + c * xq[u].y);
          }
        }
      }
      __syncthreads();
      // ---- phase 3: row rotations  A[p, :] <- c A[p, :] - s A[q, :],
      //                              A[q, :] <- conj(s) A[p, :] + c A[q, :] ----
      for (int e0 = tid; e0 < half * n; e0 += kEigThreads * kEigBatch) {
        double2 xp[kEigBatch], xq[kEigBatch];
        int off_p[kEigBatch], off_q[kEigBatch], prs[kEigBatch];
#pragma unroll
        for (int u = 0; u < kEigBatch; ++u) {
          const int e = e0 + u * kEigThreads;
          prs[u] = -1;
          if (e < half * n) {
            const int pr = e / n, j = e - pr * n;
            if (srot[pr]) {
              prs[u] = pr;
              off_p[u] = sp[pr] * n + j;
              off_q[u] = sq[pr] * n + j;
              xp[u] = A[off_p[u]];
              xq[u] = A[off_q[u]];
            }
          }
        }
#pragma unroll
        for (int u = 0; u < kEigBatch; ++u) {
          if (prs[u] >= 0) {
            const double c = sc[prs[u]];
            const double2 s = ss[prs[u]];
            const double2 t1 = cmuld(s, xq[u]), t2 = cmuld(conjd(s), xp[u]);
            A[off_p[u]] = make_double2(c * xp[u].x - t1.x, c * xp[u].y - t1.y);
            A[off_q[u]] = make_double2(t2.x + c * xq[u].x, t2.y + c * xq[u].y);
          }
        }
      }
      __syncthreads();
    }
    const int done = (nrot == 0);
    __syncthreads();
    ++sweeps_run;
    if (done) {
      converged = 1;
      break;
    }
  }
  if (tid == 0) {
    jb.status[0] = converged ? 0 : 1;
    jb.status[1] = sweeps_run;
  }

  for (int i = tid; i < n; i += kEigThreads) lam[i] = A[i * n + i].x;
  __syncthreads();
  eig_finish(n, r, tid, lam, col_of, phase, V, reinterpret_cast<float2*>(jb.U));
}

// The same solver for n <= 128 with the Hermitian work matrix held in LDS (lower triangle,
// n (n + 1) / 2 complex doubles <= 132 KB): a round is then one barrier-separated pair of phases
// on LDS - rotations from the pivots, then every 2 x 2 block (pair a, pair b), a >= b, updated in one
// step as  L_a B R_b  (the column and the row rotation of the two-pass form fused) - and only the
// eigenvector accumulator V goes through memory, once per round.
constexpr int kEigTriMaxN = 128;

__device__ __forceinline__ int tri_idx(int i, int j) { return i * (i + 1) / 2 + j; }           // i >= j
__device__ __forceinline__ double2 tri_get(const double2* T, int i, int j) {
  return i >= j ? T[tri_idx(i, j)] : conjd(T[tri_idx(j, i)]);
}
__device__ __forceinline__ void tri_put(double2* T, int i, int j, double2 v) {
  if (i >= j) T[tri_idx(i, j)] = v; else T[tri_idx(j, i)] = conjd(v);
}

__global__ __launch_bounds__(kEigThreads) void k_eig_tri(EigJobs jobs) {
  extern __shared__ double2 T[];                // lower triangle of the work matrix
  const EigJob jb = jobs.job[blockIdx.x];
  if (jb.use_fast && jb.status[2] == 0) return;   // the tridiagonal path has delivered this factor
  const int n = jb.n;
  const int tid = threadIdx.x;
  const double2* G = reinterpret_cast<const double2*>(jb.gram);
  EigLogHeader* hdr = reinterpret_cast<EigLogHeader*>(jb.A);
  RotLog* rlog = reinterpret_cast<RotLog*>(reinterpret_cast<char*>(jb.A) + sizeof(EigLogHeader));
  int nlogged = 0;                               // rounds written to the log (uniform over the block)

  __shared__ int sp[kEigTriMaxN / 2 + 1], sq[kEigTriMaxN / 2 + 1];
  __shared__ double sc[kEigTriMaxN / 2 + 1];
  __shared__ double2 ss[kEigTriMaxN / 2 + 1];
  __shared__ int srot[kEigTriMaxN / 2 + 1];
  __shared__ int nrot;
  __shared__ double red[kEigThreads];

  double tr = 0.;
  for (int e = tid; e < n * n; e += kEigThreads) {
    const int i = e / n, j = e - i * n;
    const double2 g = G[e];
    if (i >= j) T[tri_idx(i, j)] = g;
    if (i == j) tr += g.x;
  }
  red[tid] = tr;
  __syncthreads();
  for (int off = kEigThreads / 2; off > 0; off >>= 1) {
    if (tid < off) red[tid] += red[tid + off];
    __syncthreads();
  }
  const double trace = red[0];
  const double floor2 = (2.2e-18 * trace / n) * (2.2e-18 * trace / n);
  const double eps2 = 4.93e-32;
  const int m = n + (n & 1);
  const int half = m / 2;
  const int nblocks = half * (half - 1) / 2;
  // The off-pivot blocks (pair a, pair b), a > b, a thread updates in every round: e = tid, tid + 1024
  // (2016 blocks for 64 pairs: two per thread); decoded once, packed as a << 8 | b, -1 = none.  The
  // pivot block (a, a) is updated by the thread that computes its rotation.
  constexpr int kBlocksPerThread = (kEigTriMaxN / 2) * (kEigTriMaxN / 2 - 1) / 2 / kEigThreads + 1;
  int my_ab[kBlocksPerThread];
#pragma unroll
  for (int u = 0; u < kBlocksPerThread; ++u) {
    const int e = tid + u * kEigThreads;
    my_ab[u] = -1;
    if (e < nblocks) {
      int a = (int)((sqrtf(8.f * (float)e + 1.f) + 1.f) * 0.5f);
      while (a * (a - 1) / 2 > e) --a;
      while ((a + 1) * a / 2 <= e) ++a;
      my_ab[u] = (a << 8) | (e - a * (a - 1) / 2);
    }
  }
  // B <- L_a B R_b for the 2 x 2 block (rows p_a, q_a; columns p_b, q_b), L = [[c, -s], [conj(s), c]],
  // R = [[c, s], [-conj(s), c]]; a == b: the pivot block, of which the lower triangle is kept
  auto update_block = [&](int a, int b) {
    const int pa = sp[a], qa = sq[a], pb = sp[b], qb = sq[b];
    const bool qa_ok = qa < n, qb_ok = qb < n;         // padding player of an odd n: no such row / column
    const double ca = sc[a], cb = sc[b];
    const double2 sa = ss[a], sb = ss[b];
    const double2 zero = make_double2(0., 0.);
    double2 b00 = tri_get(T, pa, pb);
    double2 b01 = qb_ok ? tri_get(T, pa, qb) : zero;
    double2 b10 = qa_ok ? tri_get(T, qa, pb) : zero;
    double2 b11 = (qa_ok && qb_ok) ? tri_get(T, qa, qb) : zero;
    // rows: [r_p; r_q] <- [c r_p - s r_q; conj(s) r_p + c r_q]
    {
      const double2 t00 = cmuld(sa, b10), t01 = cmuld(sa, b11);
      const double2 u00 = cmuld(conjd(sa), b00), u01 = cmuld(conjd(sa), b01);
      const double2 n00 = make_double2(ca * b00.x - t00.x, ca * b00.y - t00.y);
      const double2 n01 = make_double2(ca * b01.x - t01.x, ca * b01.y - t01.y);
      const double2 n10 = make_double2(u00.x + ca * b10.x, u00.y + ca * b10.y);
      const double2 n11 = make_double2(u01.x + ca * b11.x, u01.y + ca * b11.y);
      b00 = n00; b01 = n01; b10 = n10; b11 = n11;
    }
    // columns: [x_p, x_q] <- [c x_p - conj(s) x_q, s x_p + c x_q]
    {
      const double2 t00 = cmuld(conjd(sb), b01), t10 = cmuld(conjd(sb), b11);
      const double2 u00 = cmuld(sb, b00), u10 = cmuld(sb, b10);
      const double2 n00 = make_double2(cb * b00.x - t00.x, cb * b00.y - t00.y);
      const double2 n10 = make_double2(cb * b10.x - t10.x, cb * b10.y - t10.y);
      const double2 n01 = make_double2(u00.x + cb * b01.x, u00.y + cb * b01.y);
      const double2 n11 = make_double2(u10.x + cb * b11.x, u10.y + cb * b11.y);
      b00 = n00; b01 = n01; b10 = n10; b11 = n11;
    }
    if (a == b) {
      T[tri_idx(pa, pa)] = b00;
      if (qa_ok) {
        T[tri_idx(qa, qa)] = b11;
        T[tri_idx(qa, pa)] = b10;
      }
    } else {
      tri_put(T, pa, pb, b00);
      if (qb_ok) tri_put(T, pa, qb, b01);
      if (qa_ok) tri_put(T, qa, pb, b10);
      if (qa_ok && qb_ok) tri_put(T, qa, qb, b11);
    }
  };

  int sweeps_run = 0, converged = 0;
  for (int sweep = 0; sweep < jb.max_sweeps; ++sweep) {
    if (tid == 0) nrot = 0;
    __syncthreads();
    for (int round = 0; round < m - 1; ++round) {
      // ---- phase 1: pairs of this round and their rotations ----
      int rot = 0;
      if (tid < half) {
        int p, q;
        jacobi_pair(tid, round, m, p, q);
        double c = 1.;
        double2 s = make_double2(0., 0.);
        if (q < n)                                     // a_pq = conj(T[q, p]) since p < q
          rot = jacobi_rotation(T[tri_idx(p, p)].x, T[tri_idx(q, q)].x, conjd(T[tri_idx(q, p)]), eps2, floor2,
                                c, s) ? 1 : 0;
        sp[tid] = p;
        sq[tid] = q;
        sc[tid] = c;
        ss[tid] = s;
        srot[tid] = rot;
        if (rot) atomicAdd(&nrot, 1);
      }
      if (!__syncthreads_or(rot)) continue;            // nothing rotates in this round (late sweeps)
      // ---- phase 2a: the round's rotations go to the log; the eigenvector accumulator is built from
      //      it afterwards by k_eig_apply, all rows in parallel ----
      if (tid < half) {
        RotLog e;
        e.c = sc[tid];
        e.sx = ss[tid].x;
        e.sy = ss[tid].y;
        e.p = srot[tid] ? sp[tid] : -1;
        e.q = sq[tid];
        rlog[(size_t)nlogged * half + tid] = e;
      }
      ++nlogged;
      // ---- phase 2b: every block (pair a, pair b), a >= b:  B <- L_a B R_b ----
      if (tid < half && srot[tid]) update_block(tid, tid);   // own pivot block (nobody else touches it)
#pragma unroll
      for (int u = 0; u < kBlocksPerThread; ++u) {
        if (my_ab[u] < 0) continue;
        const int a = my_ab[u] >> 8, b = my_ab[u] & 255;
        if (!srot[a] && !srot[b]) continue;
        update_block(a, b);
      }
      __syncthreads();
    }
    const int done = (nrot == 0);
    __syncthreads();
    ++sweeps_run;
    if (done) {
      converged = 1;
      break;
    }
  }
  for (int i = tid; i < n; i += kEigThreads) hdr->lam[i] = T[tri_idx(i, i)].x;
  if (tid == 0) {
    hdr->rounds = nlogged;
    jb.status[0] = converged ? 0 : 1;
    jb.status[1] = sweeps_run;
  }
}

// Eigenvector accumulator from the rotation log: V = R_1 R_2 ... (every round's rotations act on
// column pairs), so each ROW of V evolves on its own: one wavefront per row, the row in LDS, lane =
// slot of the round; the arithmetic per element is that of the in-kernel update of k_eig.
constexpr int kLogAhead = 4;                     // rounds whose log entries are in flight

__global__ __launch_bounds__(64) void k_eig_apply(EigJobs jobs) {
  const EigJob jb = jobs.job[blockIdx.y];
  if (jb.use_fast && jb.status[2] == 0) return;
  const int n = jb.n;
  const int row = blockIdx.x;
  if (row >= n) return;
  __shared__ double2 x[kEigTriMaxN];
  const int lane = threadIdx.x;
  for (int j = lane; j < n; j += 64) x[j] = make_double2(j == row ? 1. : 0., 0.);
  const EigLogHeader* hdr = reinterpret_cast<const EigLogHeader*>(jb.A);
  const RotLog* rlog = reinterpret_cast<const RotLog*>(reinterpret_cast<const char*>(jb.A) + sizeof(EigLogHeader));
  const int half = (n + (n & 1)) / 2;
  const int rounds = hdr->rounds;
  const int slot = lane < half ? lane : half - 1;          // idle lanes shadow the last slot, write nothing
  RotLog ahead[kLogAhead];
#pragma unroll
  for (int d = 0; d < kLogAhead; ++d) ahead[d] = rlog[(size_t)(d < rounds ? d : 0) * half + slot];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int r0 = 0; r0 < rounds; r0 += kLogAhead) {
#pragma unroll
    for (int d = 0; d < kLogAhead; ++d) {
      const int rr = r0 + d;
      const RotLog e = ahead[d];
      const int nxt = rr + kLogAhead;
      ahead[d] = rlog[(size_t)(nxt < rounds ? nxt : 0) * half + slot];
      if (rr < rounds && lane < half && e.p >= 0) {
        const double2 xp = x[e.p], xq = x[e.q];
        const double2 sc_ = make_double2(e.sx, e.sy);
        const double2 t1 = cmuld(conjd(sc_), xq), t2 = cmuld(sc_, xp);
        x[e.p] = make_double2(e.c * xp.x - t1.x, e.c * xp.y - t1.y);
        x[e.q] = make_double2(t2.x + e.c * xq.x, t2.y + e.c * xq.y);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // the next round reads what this one wrote
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
  double2* V = reinterpret_cast<double2*>(jb.V);
  for (int j = lane; j < n; j += 64) V[(size_t)row * n + j] = x[j];
}

// Ordering, phase convention and the float32 factor, from the eigenvalues in the log header and V.
__global__ __launch_bounds__(kEigThreads) void k_eig_finish(EigJobs jobs) {
  const EigJob jb = jobs.job[blockIdx.x];
  if (jb.use_fast && jb.status[2] == 0) return;
  __shared__ double lam[kEigTriMaxN];
  __shared__ int col_of[kEigTriMaxN];
  __shared__ double2 phase[kEigTriMaxN];
  const EigLogHeader* hdr = reinterpret_cast<const EigLogHeader*>(jb.A);
  for (int i = threadIdx.x; i < jb.n; i += kEigThreads) lam[i] = hdr->lam[i];
  __syncthreads();
  eig_finish(jb.n, jb.r, threadIdx.x, lam, col_of, phase, reinterpret_cast<const double2*>(jb.V),
             reinterpret_cast<float2*>(jb.U));
}

// ---------------------------------------------------------------------------------------------
// The same eigenvectors by the classical route, for n <= 128:
//   k_trid      (one workgroup per matrix) Householder tridiagonalisation  A = Q T Q^H; reflector i annihilates column
//               i below the subdiagonal; T real symmetric tridiagonal
//   k_trid_vec  (one wavefront per eigenvector)
//               the k-th largest eigenvalue of T by multisection on Sturm counts (64 points per step, from the
//               Gershgorin interval), its eigenvector by inverse iteration (Gaussian elimination
//               with partial pivoting on T - lambda I from both ends, three solves from a fixed pseudo-random vector), the
//               back-transformation with the reflectors, the phase convention and the float32 factor.
// A cyclic Jacobi sweep reads and writes the whole matrix in every one of its n - 1 rounds, about ten sweeps long;
// the tridiagonalisation touches the trailing block once per step.
// Inverse iteration separates eigenvectors only as well as their eigenvalues are separated: if an eigenvalue lies
// within 1e-7 of the spectral radius of one of the r leading ones (exactly repeated eigenvalues, a zero matrix),
// this path declines (status[2] = 1) and the Jacobi kernels, which handle clusters gracefully, solve the matrix.
//
// Everything here is a serial chain of one wavefront's instructions (4.5 cycles each, also where one needs the result of
// the one before; a sum over the lanes 156), so what counts is how many there are.  k_trid keeps the matrix in registers, passes
// one barrier per step and has the rank-2 update and the next matrix-vector product in one pass with the broadcast of rows
// inside the multiply-adds.  With two barriers, the update and the product apart and the rows' factors read from LDS a step took
// 1.7 us at n = 64 and 2.7 at 128; it takes 1.1 and 1.8.
// Measured, four modes at once, us, tridiagonalisation + vectors together: 128,128,128,65 (r 32,32,32,16) 433 -> 277;
// 64,64,32,17 (r 16,16,8,4) 155 -> 91.
constexpr double kClusterTol = 1e-7;

// work buffer of a job: reflector factors, T, and the bounds of its spectrum
__device__ __forceinline__ double2* trid_tau(const EigJob& jb) { return reinterpret_cast<double2*>(jb.A); }
__device__ __forceinline__ double* trid_d(const EigJob& jb) { return jb.A + 2 * jb.n; }
__device__ __forceinline__ double* trid_e(const EigJob& jb) { return jb.A + 3 * jb.n; }
__device__ __forceinline__ double* trid_bounds(const EigJob& jb) { return jb.A + 4 * jb.n; }   // lower, upper

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const int2 w = __builtin_bit_cast(int2, v);
  int2 r;
  r.x = __builtin_amdgcn_mov_dpp(w.x, CTRL, 0xF, 0xF, true);
  r.y = __builtin_amdgcn_mov_dpp(w.y, CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, r);
}
constexpr int kMirror16 = 0x140, kMirror8 = 0x141, kReverse4 = 0x1B, kSwap2 = 0xB1;   // lane ^ 15, ^ 7, ^ 3, ^ 1

// a, b -> (even rows of 16 lanes: a of both rows of the pair, odd rows: b of both): one step of a reduction that also
// halves the values; with a == b it adds the two rows of a pair
__device__ __forceinline__ double add_rows16(double a, double b) {
  const int2 x = __builtin_bit_cast(int2, a), y = __builtin_bit_cast(int2, b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x.x, (unsigned)y.x, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)x.y, (unsigned)y.y, false, false);
  return __builtin_bit_cast(double, make_int2((int)lo[0], (int)hi[0])) +
         __builtin_bit_cast(double, make_int2((int)lo[1], (int)hi[1]));
}
__device__ __forceinline__ double add_halves(double a) {
  const int2 x = __builtin_bit_cast(int2, a);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x.x, (unsigned)x.x, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)x.y, (unsigned)x.y, false, false);
  return __builtin_bit_cast(double, make_int2((int)lo[0], (int)hi[0])) +
         __builtin_bit_cast(double, make_int2((int)lo[1], (int)hi[1]));
}
// sum over the 64 lanes, the same bits in every lane
__device__ __forceinline__ double wave_sum_d(double v) {
  v += dpp_d<kMirror16>(v);
  v += dpp_d<kMirror8>(v);
  v += dpp_d<kReverse4>(v);
  v += dpp_d<kSwap2>(v);
  return add_halves(add_rows16(v, v));
}

// 1 / q from the hardware's reciprocal estimate and two Newton steps: a correctly rounded float64 division is four
// times as long, and no closer here (|1 - q r| <= 2^-53 for both over 2^28 arguments of every exponent between -200 and
// 200).  The pivots of the inverse iteration need less; tau and scale of a reflector, (beta - alpha) r and a complex
// conjugate times r, are each within 3 x 2^-53 of theirs, so a reflector departs from unitarity by at most some 20 x 2^-53
// and the n - 1 <= 127 of a matrix together by 3e-13: five orders below the rounding of the float32 factor.
__device__ __forceinline__ double rcp_nr(double q) {
  double r = __builtin_amdgcn_rcp(q);
  r = fma(fma(-q, r, 1.), r, r);
  r = fma(fma(-q, r, 1.), r, r);
  return r;
}

__device__ __forceinline__ uint32_t trid_mix(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7FEB352Du;
  x ^= x >> 15;
  x *= 0x846CA68Bu;
  x ^= x >> 16;
  return x;
}

// acc + S x for one row: the row's value of every operand sits in lane `LANE` of each group of 16 lanes, and the matrix
// column's in the lane's own registers.  S <- S - v w^H - w v^H first, then acc <- acc + conj(S) x (ay - az is the
// imaginary part).  Written out because the broadcast is part of the multiply-add (v_fmac_f64_dpp: 4.9 cycles, 4.5 without),
// where the compiler makes a move of each (a tridiagonalisation of 128 rows 16 % longer); s_nop 1: a DPP operand may not be
// read within two states of its last write.
template <int LANE>
__device__ __forceinline__ void trid_row(double2& s, double& ax, double& ay, double& az, const double2& v, const double2& w,
                                         const double2& x, const double2& nvc, const double2& nwc, double vcy, double wcy) {
#define TGRAD_ROW(d, src, m) "v_fmac_f64_dpp %" #d ", %" #src ", %" #m " row_newbcast:%17 row_mask:0xf bank_mask:0xf\n\t"
  asm("s_nop 1\n\t"
      TGRAD_ROW(0, 5, 13) TGRAD_ROW(1, 5, 16) TGRAD_ROW(0, 6, 14) TGRAD_ROW(1, 6, 13)      // v_j conj(w_k)
      TGRAD_ROW(0, 7, 11) TGRAD_ROW(1, 7, 15) TGRAD_ROW(0, 8, 12) TGRAD_ROW(1, 8, 11)      // w_j conj(v_k)
      TGRAD_ROW(2, 9, 0) TGRAD_ROW(3, 10, 0) TGRAD_ROW(2, 10, 1) TGRAD_ROW(4, 9, 1)        // conj(S) x_j
      : "+&v"(s.x), "+&v"(s.y), "+&v"(ax), "+&v"(ay), "+&v"(az)
      : "v"(v.x), "v"(v.y), "v"(w.x), "v"(w.y), "v"(x.x), "v"(x.y), "v"(nvc.x), "v"(nvc.y), "v"(nwc.x), "v"(nwc.y), "v"(vcy),
        "v"(wcy), "n"(LANE));
#undef TGRAD_ROW
}

// Place of row j in the LDS vectors: index rho + 4 m of a group of 64 at 16 rho + m, so that lane (rho, m) = 16 rho + m of a
// wavefront reads its row there and every group of 16 lanes a wavefront's columns.
__device__ __forceinline__ int trid_pos(int j) { return (j & 64) + 16 * (j & 3) + ((j & 63) >> 2); }

// Wavefront (ch, rg) holds columns 64 ch + rg + 4 m (m = lane % 16), lane (rho, m) of it rows 64 s + rho + 4 a, a < 16, s < NS.
// A step is one barrier long: behind it, every wavefront has column i + 1 of S as it was before reflector i and y = S x (x: what
// column i has below row i + 1), from which it derives S v = column + scale y, w and the next column z by itself, one row per
// lane; its columns' entries of v and w come from other lanes (ds_bpermute).  The rank-2 update of S and the product of the new
// S with the next column then are one pass over the registers.
struct TridLds {
  double2 col[2][kEigTriMaxN], y[2][kEigTriMaxN];   // by parity of the step: a slower wavefront still reads the other
  double d[kEigTriMaxN], e[kEigTriMaxN];
};

// Workgroup barrier that orders LDS only (a full one would also wait for the reflectors on their way to memory)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ double read_lane_d(double v, int lane) {
  const int2 w = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(w.x, lane), __builtin_amdgcn_readlane(w.y, lane)));
}
__device__ __forceinline__ double permute_d(int from, double v) {   // from: 4 x lane
  const int2 w = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_ds_bpermute(from, w.x), __builtin_amdgcn_ds_bpermute(from, w.y)));
}

template <int NS>
__device__ __forceinline__ void tridiagonalise(const EigJob& jb, TridLds& lds) {
  constexpr int T = 256 * NS;
  const int n = jb.n;
  const int tid = threadIdx.x, lane = tid & 63, rho = lane >> 4, m = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ch = wave >> 2, rg = wave & 3;
  const double2* G = reinterpret_cast<const double2*>(jb.gram);
  double2* Vg = reinterpret_cast<double2*>(jb.V);   // reflector i: Vg[i * n + row], zero up to row i
  double2* tauG = trid_tau(jb);
  const double2 zero = make_double2(0., 0.);
  const int kc = 64 * ch + rg + 4 * m, pc = 64 * ch + 16 * rg + m;   // own column, its place
  const int from = 4 * (16 * rg + m);            // the lane that has row kc, times 4
  const bool writer = rg == 1 && ch == (n > 64 ? NS - 1 : 0);   // (a wavefront that takes part to the last step)
  int jr[NS];                                    // own rows, of which a wavefront's 64 lanes have one each
#pragma unroll
  for (int s = 0; s < NS; ++s) jr[s] = 64 * s + rho + 4 * m;

  double2 S[NS][16];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int a = 0; a < 16; ++a) {
      const int row = 64 * s + rho + 4 * a;
      S[s][a] = row < n && kc < n ? G[row * n + kc] : zero;
    }
  double2 x[NS], v[NS], w[NS];                   // column i below row i + 1; reflector and w of step i - 1, by rows
  double2 vc = zero, wc = zero;                  // and by own column
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    x[s] = jr[s] > 1 && jr[s] < n ? G[jr[s] * n] : zero;
    v[s] = w[s] = zero;
  }
  double2 alpha = n > 1 ? G[n] : zero;           // entry i + 1 of column i
  double diag = G[0].x;
  for (int j = tid; j < 2 * kEigTriMaxN; j += T) (&lds.col[0][0])[j] = (&lds.y[0][0])[j] = zero;   // (places past n stay zero)
  __syncthreads();

  // Steps i0 .. i1 - 1, of which rows and columns below 64 s0 are finished.  Every multiply-add is written out: what the
  // wavefronts derive from the LDS vectors each for itself has to have the same bits.
  auto steps = [&](int i0, int i1, auto s0_c) __attribute__((always_inline)) {
    constexpr int s0 = decltype(s0_c)::value;
    if (ch < s0 || 64 * ch >= n) {               // nothing left of this wavefront's columns
      for (int i = i0; i < i1; ++i) lds_barrier();
      return;
    }
    for (int i = i0; i < i1; ++i) {
      const int par = i & 1;
      // the reflector of column i: v = (0 .. 0, 1, scale x)
      double xn2 = 0.;
#pragma unroll
      for (int s = s0; s < NS; ++s) xn2 = fma(x[s].x, x[s].x, fma(x[s].y, x[s].y, xn2));
      xn2 = wave_sum_d(xn2);
      double2 tau = zero, scale = zero;
      double beta = alpha.x;
      if (!(xn2 == 0. && alpha.y == 0.)) {
        // beta = -+ sqrt(t), 1 / beta: the hardware's reciprocal root and two Newton steps
        const double t = fma(alpha.x, alpha.x, fma(alpha.y, alpha.y, xn2));
        double r = __builtin_amdgcn_rsq(t);
        r = fma(0.5 * r, fma(-t * r, r, 1.), r);
        r = fma(0.5 * r, fma(-t * r, r, 1.), r);
        const double root = t * r;
        beta = -copysign(fma(fma(-root, root, t), 0.5 * r, root), alpha.x);
        const double inv_beta = -copysign(r, alpha.x);
        tau = make_double2((beta - alpha.x) * inv_beta, -alpha.y * inv_beta);
        const double2 z = make_double2(alpha.x - beta, alpha.y);              // 1 / (alpha - beta)
        const double inv = rcp_nr(fma(z.x, z.x, z.y * z.y));
        scale = make_double2(z.x * inv, -z.y * inv);
      }
      double2 vn[NS];
#pragma unroll
      for (int s = s0; s < NS; ++s) {
        vn[s].x = jr[s] == i + 1 ? 1. : fma(scale.x, x[s].x, -(scale.y * x[s].y));
        vn[s].y = fma(scale.x, x[s].y, scale.y * x[s].x);
      }
      const double2 vo = NS > 1 && s0 == 0 && ch > 0 ? vn[NS - 1] : vn[s0];
      const double2 vnc = make_double2(permute_d(from, vo.x), permute_d(from, vo.y));
      if (writer) {
        if (lane == 0) {
          lds.d[i] = diag;
          lds.e[i] = beta;
          tauG[i] = tau;
        }
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (jr[s] < n) Vg[(size_t)i * n + jr[s]] = s < s0 ? zero : vn[s];
      }
      double ax = 0., ay = 0., az = 0.;
      const double2 nvc = make_double2(-vc.x, -vc.y), nwc = make_double2(-wc.x, -wc.y);
#pragma unroll
      for (int s = s0; s < NS; ++s) {
        auto group = [&](auto g_c) __attribute__((always_inline)) {          // 16 rows: all finished, or past the matrix
          constexpr int g = decltype(g_c)::value;
          if (64 * s + 16 * g + 16 <= i + 1 || 64 * s + 16 * g >= n) return;
          trid_row<4 * g>(S[s][4 * g], ax, ay, az, v[s], w[s], x[s], nvc, nwc, vc.y, wc.y);
          trid_row<4 * g + 1>(S[s][4 * g + 1], ax, ay, az, v[s], w[s], x[s], nvc, nwc, vc.y, wc.y);
          trid_row<4 * g + 2>(S[s][4 * g + 2], ax, ay, az, v[s], w[s], x[s], nvc, nwc, vc.y, wc.y);
          trid_row<4 * g + 3>(S[s][4 * g + 3], ax, ay, az, v[s], w[s], x[s], nvc, nwc, vc.y, wc.y);
          if ((i + 1) >> 4 == 4 * s + g) {       // row i + 1 is column i + 1, conjugated
            const int q = (i + 1) & 12;
            const double2 lo = q & 4 ? S[s][4 * g + 1] : S[s][4 * g], hi = q & 4 ? S[s][4 * g + 3] : S[s][4 * g + 2];
            const double2 r = q & 8 ? hi : lo;
            if (rho == ((i + 1) & 3)) lds.col[par][pc] = make_double2(r.x, -r.y);
          }
        };
        group(std::integral_constant<int, 0>());
        group(std::integral_constant<int, 1>());
        group(std::integral_constant<int, 2>());
        group(std::integral_constant<int, 3>());
      }
      const double y = add_halves(add_rows16(ax, ay - az));                  // even rows of lanes: its real part, odd: imaginary
      if (rho < 2) reinterpret_cast<double*>(&lds.y[par][pc])[rho] = y;
      lds_barrier();
      // w = tau S v - 1/2 |tau|^2 (v^H S v) v;   S <- S - v w^H - w v^H, of which z is column i + 1
      double2 c[NS], q[NS];
      double dot = 0.;
#pragma unroll
      for (int s = s0; s < NS; ++s) {
        c[s] = lds.col[par][64 * s + lane];
        const double2 yl = lds.y[par][64 * s + lane];
        q[s].x = fma(scale.x, yl.x, fma(-scale.y, yl.y, c[s].x));
        q[s].y = fma(scale.x, yl.y, fma(scale.y, yl.x, c[s].y));
        v[s] = vn[s];
        dot = fma(v[s].x, q[s].x, fma(v[s].y, q[s].y, dot));
      }
      vc = vnc;
      const double alpha2 = -0.5 * fma(tau.x, tau.x, tau.y * tau.y) * wave_sum_d(dot);
#pragma unroll
      for (int s = s0; s < NS; ++s) {
        const bool in = jr[s] > i;               // (finished rows of the LDS vectors are stale)
        w[s].x = in ? fma(alpha2, v[s].x, fma(tau.x, q[s].x, -(tau.y * q[s].y))) : 0.;
        w[s].y = in ? fma(alpha2, v[s].y, fma(tau.x, q[s].y, tau.y * q[s].x)) : 0.;
      }
      const double2 wo = NS > 1 && s0 == 0 && ch > 0 ? w[NS - 1] : w[s0];
      wc = make_double2(permute_d(from, wo.x), permute_d(from, wo.y));
      // entry j of the vector t, which every wavefront has
      auto entry = [&](const double2 (&t)[NS], int j) -> double2 {
        const int at = trid_pos(j) & 63;
        if (NS > 1 && s0 == 0 && j >= 64) return make_double2(read_lane_d(t[NS - 1].x, at), read_lane_d(t[NS - 1].y, at));
        return make_double2(read_lane_d(t[s0].x, at), read_lane_d(t[s0].y, at));
      };
      const double2 w1 = entry(w, i + 1);
      double2 z[NS];
#pragma unroll
      for (int s = s0; s < NS; ++s) {
        z[s].x = fma(-v[s].x, w1.x, fma(-v[s].y, w1.y, c[s].x - w[s].x));
        z[s].y = fma(-v[s].y, w1.x, fma(v[s].x, w1.y, c[s].y - w[s].y));
        x[s].x = jr[s] > i + 2 ? z[s].x : 0.;
        x[s].y = jr[s] > i + 2 ? z[s].y : 0.;
      }
      diag = entry(z, i + 1).x;
      alpha = entry(z, i + 2 < 64 * NS ? i + 2 : i + 1);
    }
  };
  // step 63 has column 63 behind it: entries of its z below row 64 are not read any more
  steps(0, NS > 1 && n > 64 ? 63 : n - 1, std::integral_constant<int, 0>());
  if constexpr (NS > 1)
    if (n > 64) steps(63, n - 1, std::integral_constant<int, 1>());
  if (writer && lane == 0) {
    lds.d[n - 1] = diag;
    lds.e[n - 1] = 0.;
  }
  __syncthreads();
  for (int i = tid; i < n; i += T) {
    trid_d(jb)[i] = lds.d[i];
    trid_e(jb)[i] = lds.e[i];
  }
  if (wave == 0) {                               // Gershgorin interval
    double lo = 1e300, hi = -1e300;
    for (int i = lane; i < n; i += 64) {
      const double rad = (i > 0 ? fabs(lds.e[i - 1]) : 0.) + (i + 1 < n ? fabs(lds.e[i]) : 0.);
      lo = fmin(lo, lds.d[i] - rad);
      hi = fmax(hi, lds.d[i] + rad);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      lo = fmin(lo, __shfl_xor(lo, off, 64));
      hi = fmax(hi, __shfl_xor(hi, off, 64));
    }
    if (lane == 0) {
      const double slack = 2.1 * fmax(fabs(lo), fabs(hi)) * 2.220446049250313e-16 * n;
      trid_bounds(jb)[0] = lo - slack;
      trid_bounds(jb)[1] = hi + slack;
      jb.status[0] = 0;
      jb.status[1] = 0;
      jb.status[2] = 0;                          // k_trid_vec declines
    }
  }
}

// One workgroup per matrix.  NS: groups of 64 rows.
template <int NS>
__global__ __launch_bounds__(256 * NS) __attribute__((amdgpu_waves_per_eu(NS, NS))) void k_trid(EigJobs jobs) {
  __shared__ TridLds lds;
  tridiagonalise<NS>(jobs.job[blockIdx.x], lds);
}

// Eigenvector k of job blockIdx.y.  T is scaled by a power of two so that its spectral radius lies in [1, 2).
// Sturm counts without divisions: p_(i+1) = (d_i - x) p_i - e_(i-1)^2 p_(i-1), one sign change per eigenvalue below x;
// the chain is one multiply-add per row (a quotient recurrence has a reciprocal in it).  Every eighth row the pair is
// brought back to order one; e^2 has a floor of 1e-60 so that no two consecutive p vanish: a pair then shrinks by at most
// 1e-240 between two such rows.
// Six steps leave the eigenvalue in an interval of 4 / (65^5 64) < 6e-11 of the scaled T.  Inverse iteration needs no more: an
// eigenvalue at least kClusterTol away loses a factor of 3e-4 or more against it in each of the three solves, 2e-11 together,
// and the vector that they converge to is that of T, not of the shift.  (Ten steps, to the last bit of the eigenvalue, leave
// factors equally far from 64 bits: rms 6.3e-9, 3.2e-9 and 2.2e-9 at 16, 64 and 128 rows with either, leading pairs 1.2e-7, 2e-7, 4e-7
// and 2e-6 of the radius apart.)
constexpr int kMultiSteps = 6;
constexpr int kAheadRefl = 12;
constexpr int kSideRows = kEigTriMaxN / 2 + 8;   // rows of one side, and what is read ahead of them

__global__ __launch_bounds__(64) void k_trid_vec(EigJobs jobs) {
  const EigJob jb = jobs.job[blockIdx.y];
  const int n = jb.n, r = jb.r;
  const int k = blockIdx.x;
  if (k >= r) return;
  const int lane = threadIdx.x;
  const int r0 = lane, r1 = lane + 64;
  __shared__ double2 de[kEigTriMaxN + 24];       // (d_i, e_(i-1)^2), scaled; past n: rows that change no sign
  __shared__ double2 sde[2][kSideRows];          // (d, e towards the next row) in the order of each side
  __shared__ double2 slu[2][kSideRows][2];       // (1 / pivot, first super-diagonal), (second, multiplier)
  __shared__ double sy[2][kSideRows], sz[2][kSideRows];
  __shared__ double2 stau[kEigTriMaxN];
  const double2* tauG = trid_tau(jb);
  const double* dG = trid_d(jb);
  const double* eG = trid_e(jb);
  // everything that the wavefront reads is requested together
  const int q0 = r0 < n ? r0 : n - 1, q1 = r1 < n ? r1 : n - 1;
  const double gl = trid_bounds(jb)[0], gu = trid_bounds(jb)[1];
  const double d0 = dG[q0], d1 = dG[q1], e0 = eG[q0], e1 = eG[q1], f0 = eG[q0 > 0 ? q0 - 1 : 0], f1 = eG[q1 > 0 ? q1 - 1 : 0];
  const double2 tau0 = tauG[q0], tau1 = tauG[q1];
  const double tn = fmax(fabs(gl), fabs(gu));
  // the first reflectors of the back-transformation go in flight: unconditional loads, so that no wait stands at the end of a
  // branch; a lane without a row takes row 0, where every reflector is zero
  const double2* V0 = reinterpret_cast<const double2*>(jb.V) + (r0 < n ? r0 : 0);
  const double2* V1 = reinterpret_cast<const double2*>(jb.V) + (r1 < n ? r1 : 0);
  double2 pv0[kAheadRefl], pv1[kAheadRefl];
  auto issue = [&](int i, int slot) {
    const size_t at = (size_t)(i >= 0 ? i : 0) * n;
    pv0[slot] = V0[at];
    if (n > 64) pv1[slot] = V1[at];
  };
#pragma unroll
  for (int d = 0; d < kAheadRefl; ++d) issue(n - 2 - d, d);
  if (!(tn > 0.) || !(tn <= 1e300) || gl != gl || gu != gu) {            // zero matrix, inf or NaN
    if (lane == 0) jb.status[2] = 1;
    return;
  }
  const int ex = -ilogb(tn);
  auto scaled = [&](double v) { return ldexp(v, ex); };
  const int mt = (n - 1) >> 1, mb = n - 2 - mt;  // rows eliminated from the top and from the bottom: mb is mt or one less
  auto place = [&](int row, double d, double e, double f, double2 tau) {
    const double ep = row > 0 ? scaled(f) : 0.;
    if (row < n) {
      de[row] = make_double2(scaled(d), fmax(ep * ep, 1e-60));
      stau[row] = tau;
      if (row < kSideRows) sde[0][row] = make_double2(scaled(d), row < n - 1 ? scaled(e) : 0.);
      if (n - 1 - row < kSideRows) sde[1][n - 1 - row] = make_double2(scaled(d), ep);
    } else if (row < kEigTriMaxN + 24) {
      de[row] = make_double2(8., 0.);            // d - x > 0 and e = 0: p keeps its sign
    }
  };
  place(r0, d0, e0, f0, tau0);
  place(r1, d1, e1, f1, tau1);
  place(lane + 128, 0., 0., 0., tau0);
  __syncthreads();
  auto sturm_count = [&](double x) -> int {      // eigenvalues below x
    double p0 = 0., p1 = 1.;
    int c = 0;
    uint32_t signs = 0u;                         // of the last rows, the newest in bit 0
    auto rows = [&](const double2 (&t)[8]) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double p2 = fma(t[u].x - x, p1, -(t[u].y * p0));
        signs = __builtin_amdgcn_alignbit(signs, (uint32_t)__double2hiint(p2), 31);
        p0 = p1;
        p1 = p2;
      }
      c += __popc((signs ^ (signs >> 1)) & 0xFFu);
      const int e = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
      p0 = ldexp(p0, e);
      p1 = ldexp(p1, e);
    };
    double2 t[8], u[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) t[j] = de[j];
    for (int i0 = 0; i0 < n; i0 += 16) {         // (up to 15 rows past n, of those that change no sign)
#pragma unroll
      for (int j = 0; j < 8; ++j) u[j] = de[i0 + 8 + j];
      rows(t);
#pragma unroll
      for (int j = 0; j < 8; ++j) t[j] = de[i0 + 16 + j];
      rows(u);
    }
    return c;
  };
  const double tnorm = scaled(tn);
  const int kasc = n - 1 - k;                    // k-th largest = kasc-th smallest (0-based)
  double lo = scaled(gl), hi = scaled(gu);
  bool apart = true;
  for (int step = 0; step < kMultiSteps; ++step) {
    const bool last = step == kMultiSteps - 1;
    const double h = (hi - lo) * (last ? 1. / 64. : 1. / 65.);           // (one point less in the last step)
    // the last lane of the last step looks whether the next eigenvalue (also the one behind the last kept one) is separated
    const double x = last && lane == 63 ? 0.5 * (lo + hi) - kClusterTol * tnorm : lo + (lane + 1) * h;
    const int c = sturm_count(x);
    uint64_t bal = __ballot(c > kasc);           // more than kasc eigenvalues below the point
    if (last) {
      bal &= ~0ull >> 1;
      apart = k + 1 >= n || __builtin_amdgcn_readlane(c, 63) == kasc;
    }
    const int points = last ? 63 : 64;
    const int jf = bal ? __builtin_ctzll(bal) : points;                  // the eigenvalue lies below point jf and not below jf - 1
    const double nlo = jf == 0 ? lo : lo + jf * h;
    const double nhi = jf == points ? hi : lo + (jf + 1) * h;
    lo = nlo;
    hi = nhi;
  }
  const double lam = 0.5 * (lo + hi);
  if (!(fabs(lam) <= 1e300) || !apart) {
    if (lane == 0) jb.status[2] = 1;
    return;
  }

  // ---- inverse iteration: a serial chain, so it burns at both ends: lane 0 eliminates from the first row down, lane 32 from
  // the last row up (the same code on the reversed matrix), a 2 x 2 system is left in the middle, and the substitution runs
  // outwards on both sides.  Only these two lanes are active: their writes need no predicate. ----
  const double tol = 2.220446049250313e-16 * tnorm;
  const int side = lane >> 5;
  const bool worker = (lane & 31) == 0;
  const int mh = side ? mb : mt;                 // rows eliminated from this side
  auto clamped = [&](double p) -> double { return fabs(p) < tol ? copysign(tol, p) : p; };
  uint64_t swaps = 0ull;                         // bit j: rows interchanged at step j (mt <= 63)
  double ca = 0., cu = 0.;                       // the side's last row: ca x[mh] + cu x[mh + 1]
  if (worker) {
    const double2* in = sde[side];
    double a = in[0].x - lam, du = in[0].y, sub = du;
    double2 nx = in[1];
    auto step = [&](int j) __attribute__((always_inline)) {              // elimination with partial pivoting
      const double2 ahead = in[j + 2];
      const double dn = nx.x - lam, en = nx.y;
      const bool swap = fabs(a) < fabs(sub);
      const double rp = rcp_nr(clamped(swap ? sub : a));
      const double f = (swap ? a : sub) * rp;
      slu[side][j][0] = make_double2(rp, swap ? dn : du);
      slu[side][j][1] = make_double2(swap ? en : 0., f);
      swaps |= swap ? 1ull << j : 0ull;
      a = swap ? fma(-f, dn, du) : fma(-f, du, dn);
      du = swap ? -f * en : en;
      sub = en;
      nx = ahead;
    };
    for (int j = 0; j < mb; ++j) step(j);
    if (mb < mt && side == 0) step(mb);
    ca = a;
    cu = du;
  }
  // the middle: (top row) a1 xp + u1 xq = y1, (bottom row) u2 xp + a2 xq = y2, with pivoting
  const double a1 = read_lane_d(ca, 0), u1 = read_lane_d(cu, 0), a2 = read_lane_d(ca, 32), u2 = read_lane_d(cu, 32);
  const bool mswap = fabs(a1) < fabs(u2);
  const double mp = mswap ? u2 : a1, mu = mswap ? a2 : u1;               // the pivot row
  const double mrp = rcp_nr(clamped(mp));
  const double mf = (mswap ? a1 : u2) * mrp;
  const double mrq = rcp_nr(clamped((mswap ? u1 : a2) - mf * mu));
  auto start = [&](int i) -> double {
    const uint32_t u = trid_mix((uint32_t)i * 0x9E3779B9u + (uint32_t)k * 0x85EBCA6Bu + 0x1234567u);
    return (double)u * (1. / 2147483648.) - 1.;
  };
  // place of a row in the arrays of the sides
  const int i0 = r0 <= mt ? r0 : kSideRows + n - 1 - r0, i1 = r1 <= mt ? r1 : kSideRows + n - 1 - r1;
  double* yrow = &sy[0][0];
  double* zrow = &sz[0][0];
  double z0 = 0., z1 = 0.;
  for (int it = 0; it < 3; ++it) {
    __syncthreads();                             // (one wavefront: orders the LDS accesses)
    double y = 0.;
    if (it == 0) {                               // the first right-hand side is taken as already eliminated
      if (r0 < n) yrow[i0] = start(r0);
      if (r1 < n) yrow[i1] = start(r1);
      y = start(side ? n - 1 - mh : mh);
    } else {
      if (r0 < n) zrow[i0] = z0;
      if (r1 < n) zrow[i1] = z1;
      __syncthreads();
      if (worker) {                              // elimination of the right-hand side, operands four rows ahead
        y = sz[side][0];
        auto step = [&](int j, double f, double rhs) __attribute__((always_inline)) {
          const bool swap = (swaps >> j) & 1ull;
          const double keep = swap ? rhs : y, other = swap ? y : rhs;
          sy[side][j] = keep;
          y = fma(-f, keep, other);
        };
        double f[4], rhs[4];
        auto fetch = [&](int j) __attribute__((always_inline)) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            f[u] = slu[side][j + u][1].y;
            rhs[u] = sz[side][j + u + 1];
          }
        };
        fetch(0);
        int j = 0;
        for (; j + 4 <= mb; j += 4) {
          double f0[4], h0[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            f0[u] = f[u];
            h0[u] = rhs[u];
          }
          fetch(j + 4);
#pragma unroll
          for (int u = 0; u < 4; ++u) step(j + u, f0[u], h0[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (j + u < mh) step(j + u, f[u], rhs[u]);
      }
    }
    __syncthreads();
    const double y1 = read_lane_d(y, 0), y2 = read_lane_d(y, 32);
    const double yp = mswap ? y2 : y1, yq = mswap ? y1 : y2;
    const double xq = (yq - mf * yp) * mrq, xp = (yp - mu * xq) * mrp;
    if (worker) {
      double zn1 = side ? xq : xp, zn2 = side ? xp : xq;
      sz[side][mh] = zn1;
      auto step = [&](int j, double2 p, double s2, double yi) __attribute__((always_inline)) {   // back substitution, outwards
        const double z = fma(-p.y, zn1, fma(-s2, zn2, yi)) * p.x;
        sz[side][j] = z;
        zn2 = zn1;
        zn1 = z;
      };
      const int full = mb & ~3;                  // down to a multiple of four row by row, then four at a time
#pragma unroll
      for (int u = 3; u >= 0; --u)
        if (full + u < mh) step(full + u, slu[side][full + u][0], slu[side][full + u][1].x, sy[side][full + u]);
      double2 p[4];
      double s2[4], yi[4];
      auto fetch = [&](int j) __attribute__((always_inline)) {
        const int at = j > 0 ? j : 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          p[u] = slu[side][at + u][0];
          s2[u] = slu[side][at + u][1].x;
          yi[u] = sy[side][at + u];
        }
      };
      fetch(full - 4);
      for (int j = full - 4; j >= 0; j -= 4) {
        double2 p0[4];
        double t0[4], w0[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          p0[u] = p[u];
          t0[u] = s2[u];
          w0[u] = yi[u];
        }
        fetch(j - 4);
#pragma unroll
        for (int u = 3; u >= 0; --u) step(j + u, p0[u], t0[u], w0[u]);
      }
    }
    __syncthreads();
    z0 = r0 < n ? zrow[i0] : 0.;
    z1 = r1 < n ? zrow[i1] : 0.;
    const double size = wave_sum_d(fabs(z0) + fabs(z1));                 // back to order one, by a power of two
    const int e = size > 0. && size <= 1.7e308 ? -__builtin_amdgcn_frexp_exp(size) : 0;
    z0 = ldexp(z0, e);
    z1 = ldexp(z1, e);
  }
  const double nrm2 = wave_sum_d(z0 * z0 + z1 * z1);
  const double inv = nrm2 > 0. ? rsqrt(nrm2) : 0.;

  // ---- U[:, k] = H_0 H_1 .. H_(n-2) z, the reflectors read kAheadRefl ahead; both parts of v^H x in one reduction ----
  double2 x0 = make_double2(z0 * inv, 0.), x1 = make_double2(z1 * inv, 0.);
  auto back = [&](auto two_c) __attribute__((always_inline)) {
    constexpr bool two = decltype(two_c)::value;
    for (int base = n - 2; base >= 0; base -= kAheadRefl) {
#pragma unroll
      for (int d = 0; d < kAheadRefl; ++d) {
        const int i = base - d;
        const double2 v0 = pv0[d], v1 = two ? pv1[d] : make_double2(0., 0.);
        issue(i - kAheadRefl, d);
        if (i < 0) continue;
        const double2 tau = stau[i];
        double tx = fma(v0.x, x0.x, v0.y * x0.y), ty = fma(v0.x, x0.y, -(v0.y * x0.x));
        if (two) {
          tx = fma(v1.x, x1.x, fma(v1.y, x1.y, tx));
          ty = fma(v1.x, x1.y, fma(-v1.y, x1.x, ty));
        }
        double t = add_halves(add_rows16(tx, ty));                       // even rows of lanes: real part, odd: imaginary
        t += dpp_d<kMirror16>(t);
        t += dpp_d<kMirror8>(t);
        t += dpp_d<kReverse4>(t);
        t += dpp_d<kSwap2>(t);
        const int2 w = __builtin_bit_cast(int2, t);
        const auto plo = __builtin_amdgcn_permlane16_swap((unsigned)w.x, (unsigned)w.x, false, false);
        const auto phi = __builtin_amdgcn_permlane16_swap((unsigned)w.y, (unsigned)w.y, false, false);
        const double dx = __builtin_bit_cast(double, make_int2((int)plo[0], (int)phi[0]));
        const double dy = __builtin_bit_cast(double, make_int2((int)plo[1], (int)phi[1]));
        const double2 sfac = cmuld(tau, make_double2(dx, dy));
        x0.x = fma(-sfac.x, v0.x, fma(sfac.y, v0.y, x0.x));
        x0.y = fma(-sfac.x, v0.y, fma(-sfac.y, v0.x, x0.y));
        if (two) {
          x1.x = fma(-sfac.x, v1.x, fma(sfac.y, v1.y, x1.x));
          x1.y = fma(-sfac.x, v1.y, fma(-sfac.y, v1.x, x1.y));
        }
      }
    }
  };
  if (n > 64) back(std::integral_constant<bool, true>());
  else back(std::integral_constant<bool, false>());
  // unit phase that makes the largest-modulus entry (lowest row on ties) real and positive
  double best = r0 < n ? x0.x * x0.x + x0.y * x0.y : -1.;
  int brow = r0;
  double2 bval = x0;
  {
    const double a1 = r1 < n ? x1.x * x1.x + x1.y * x1.y : -1.;
    if (a1 > best) { best = a1; brow = r1; bval = x1; }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double ob = __shfl_xor(best, off, 64);
    const int orow = __shfl_xor(brow, off, 64);
    const double ovx = __shfl_xor(bval.x, off, 64), ovy = __shfl_xor(bval.y, off, 64);
    if (ob > best || (ob == best && orow < brow)) { best = ob; brow = orow; bval = make_double2(ovx, ovy); }
  }
  const double mag = sqrt(best);
  const double2 ph = mag > 0. ? make_double2(bval.x / mag, -bval.y / mag) : make_double2(1., 0.);
  float2* U = reinterpret_cast<float2*>(jb.U);
  if (r0 < n) {
    const double2 v = cmuld(x0, ph);
    U[(size_t)r0 * r + k] = make_float2((float)v.x, (float)v.y);
  }
  if (r1 < n) {
    const double2 v = cmuld(x1, ph);
    U[(size_t)r1 * r + k] = make_float2((float)v.x, (float)v.y);
  }
}

__global__ void k_identity_factor(float2* U, int n) {
  int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n * n) U[e] = make_float2((e / n) == (e % n) ? 1.f : 0.f, 0.f);
}

}  // namespace

// Bytes of the per-mode work buffer `work_a` of launch_eig_batch: the work matrix for the
// memory-resident solver, header + rotation log (every round of every sweep) for the LDS solver.
size_t eig_work_bytes(int n) {
  if (n > kEigTriMaxN) return (size_t)n * n * sizeof(double2);
  const int m = n + (n & 1);
  return sizeof(EigLogHeader) + (size_t)kEigMaxSweeps * (m - 1) * (m / 2) * sizeof(RotLog);
}

// Tile rows that k_gram128 holds for an extent (0: the kernel for larger extents), 16 RT + 1 included where that
// row is done by vector arithmetic.  Its lane offsets reach two leading indices ahead: 2 In B elements of at most 8 bytes.
static int gram_rows(int In, int64_t B) {
  if (In > kSuper || (int64_t)In * B >= ((int64_t)1 << 28)) return 0;
  return In <= 17 ? 1 : In <= 33 ? 2 : In <= 65 ? 4 : 8;
}
static int64_t gram_tiles(int64_t A, int In, int64_t B) {
  const int rt = gram_rows(In, B), tc = rt ? gram_cols(rt) : kTC;
  return (A * B + tc - 1) / tc;
}

// All modes of up to 128 entries in one launch: their staged tiles, each as long as it takes, one after the other on a line
// of which every one of 256 workgroups (a compute unit holds one) has an equal part; where a part begins or ends inside a mode is
// a chunk of it, with a partial sum of its own.  Longer modes have a launch each, of equal chunks.
// Lengths in 0.1 us, measured by 256 workgroups of 1 to 16 tiles each; `lead` is the first round trip of a part and its partial
// sum, which a workgroup with parts of two modes has twice.  Refreshes, us, before (two chunks per compute unit, dealt by work and
// rounded to whole tiles in each mode) / now: 64x64x32x17 242 / 218, 128x128x32x17 796 / 605, 64x64x64x33 529 / 369,
// 90x77x45x23 628 / 488; a launch per mode and its reduction, 128x128x128x65: 4564 / 4514.
struct GramCost {
  uint32_t tile, lead;
};
static GramCost gram_cost(int rt, int In) {
  const int ntr = (In + 15) / 16, tiles = ntr * (ntr + 1) / 2;
  const bool tail = In == 16 * rt + 1;
  if (rt == 8) return {14u + 12u * (uint32_t)((tiles + 7) / 8), 70u};
  if (rt == 4) return {tail ? 54u : ntr == 3 ? 33u : 47u, 50u};
  if (rt == 2) return {tail ? 40u : 33u, 25u};
  return {tail ? 32u : 27u, 15u};
}

// The line of `njobs` modes, cut for `groups` workgroups.
static void gram_line(int njobs, const int64_t* A, const int* In, const int64_t* B, int groups, GramJobs* jobs) {
  uint64_t total = 0, tiles_all = 0;
  jobs->njobs = njobs;
  for (int i = 0; i < njobs; ++i) tiles_all += (uint64_t)gram_tiles(A[i], In[i], B[i]);
  // lengths are brought down until the line fits in 32 bits; where every tile has a workgroup, all are of length one
  for (int shift = tiles_all <= (uint64_t)groups ? 31 : 0; ; ++shift) {
    total = 0;
    for (int i = 0; i < njobs; ++i) {
      GramJob& jb = jobs->job[i];
      jb.rt = gram_rows(In[i], B[i]);
      const GramCost c = gram_cost(jb.rt, In[i]);
      jb.In = In[i];
      jb.A = A[i];
      jb.B = B[i];
      jb.weight = (c.tile >> shift) > 0 ? c.tile >> shift : 1u;
      jb.tiles = (uint32_t)gram_tiles(A[i], In[i], B[i]);
      if (i > 0) total += c.lead >> shift;
      jb.start = (uint32_t)total;
      total += (uint64_t)jb.tiles * jb.weight;
    }
    if (total < 0x7FFFFFFFull || shift >= 31) break;
  }
  jobs->per = (uint32_t)(total / (uint64_t)groups);
  jobs->rem = (uint32_t)(total % (uint64_t)groups);
  auto owner = [&](uint64_t at) -> int {             // the workgroup whose part holds position `at`
    const uint64_t head = (uint64_t)jobs->rem * (jobs->per + 1ull);
    return (int)(at < head ? at / (jobs->per + 1ull) : jobs->rem + (at - head) / (jobs->per ? jobs->per : 1u));
  };
  for (int i = 0; i < njobs; ++i) {
    const GramJob& jb = jobs->job[i];
    jobs->first[i] = owner(jb.start);
    jobs->nchunks[i] = owner(jb.start + (uint64_t)(jb.tiles - 1) * jb.weight) - jobs->first[i] + 1;
  }
}

// Whether a mode shares its launch with others.
bool gram_shared(int In, int64_t B) { return gram_rows(In, B) != 0; }

// Chunks of every mode of a tensor, those that share a launch first; returns the workgroups of that launch.  `room`: bytes of the
// partial sums, which are those of 512 chunks dealt by work, but not more than 256 of the mode whose are largest (with more than
// 16.8 M numbers, or one mode: these).  A launch of 256 workgroups seldom comes near; where it would, it has fewer.
int gram_num_chunks(int njobs, const int64_t* A, const int* In, const int64_t* B, int* nchunks, size_t* room) {
  const bool by_work = njobs > 1 && A[0] * In[0] * B[0] <= (int64_t)256 * 16 * 4096;
  double largest = 0., work = 0., sum = 0.;
  int64_t tiles_all = 0;
  int together = 0;
  auto most = [&](int i) -> int {
    const int64_t tiles = gram_tiles(A[i], In[i], B[i]);
    return tiles < 256 ? (tiles < 1 ? 1 : (int)tiles) : 256;
  };
  auto cost = [&](int i) -> double {
    const int rt = gram_rows(In[i], B[i]);
    return (double)gram_tiles(A[i], In[i], B[i]) * (rt == 8 ? 3. : rt == 4 ? 1.7 : 1.);
  };
  for (int i = 0; i < njobs; ++i) work += cost(i);
  for (int i = 0; i < njobs; ++i) {
    nchunks[i] = most(i);
    if (by_work) {
      const int share = (int)(512. * cost(i) / work + 0.5);
      nchunks[i] = share < 1 ? 1 : share < nchunks[i] ? share : nchunks[i];
    }
    const double n2 = (double)In[i] * In[i];
    largest = fmax(largest, (by_work ? fmin((double)((A[i] * B[i] + 15) / 16), 256.) : (double)nchunks[i]) * n2);
    sum += nchunks[i] * n2;
    if (gram_shared(In[i], B[i])) {
      ++together;
      tiles_all += gram_tiles(A[i], In[i], B[i]);
    }
  }
  double bound = largest;
  if (by_work) {
    const double part = sum > largest ? largest / sum : 1.;
    bound = 0.;
    for (int i = 0; i < njobs; ++i) {
      if (part < 1.) nchunks[i] = (int)fmax(1., (int)(nchunks[i] * part));
      bound += (double)nchunks[i] * In[i] * In[i];
    }
  }
  int groups = 0;
  if (together > 0) {
    GramJobs jobs;
    groups = tiles_all < 256 ? (int)(tiles_all < 1 ? 1 : tiles_all) : 256;
    for (;; --groups) {
      gram_line(together, A, In, B, groups, &jobs);
      sum = 0.;
      for (int i = 0; i < together; ++i) sum += (double)jobs.nchunks[i] * In[i] * In[i];
      if (sum <= bound || groups == 1) break;
    }
    for (int i = 0; i < together; ++i) nchunks[i] = jobs.nchunks[i];
    bound = fmax(bound, sum);
  }
  *room = (size_t)bound * sizeof(double2);
  return groups;
}

// Partial Grams of the modes that share a launch of `groups` workgroups, or of one that does not, in nchunks[0] chunks.
void launch_gram_batch(hipStream_t s, int njobs, const void* g, int dtype, const uint32_t* mask, const int64_t* A,
                       const int* In, const int64_t* B, int groups, const int* nchunks, double* const* partials) {
  if (!gram_shared(In[0], B[0])) {
    const int64_t tiles = (A[0] * B[0] + kTC - 1) / kTC, per = (tiles + nchunks[0] - 1) / nchunks[0] * kTC;
    const int nsup = (In[0] + kSuper - 1) / kSuper;
    const size_t lds = (size_t)2 * kSuper * kRowD * sizeof(double);     // 132 KB: more than the default limit
    const dim3 grid((unsigned)nchunks[0], (unsigned)(nsup * nsup)), block(kGramThreads);
    if (dtype == TGRAD_C64) {
      allow_lds(k_gram<TGRAD_C64>, lds);
      k_gram<TGRAD_C64><<<grid, block, lds, s>>>(g, mask, A[0], In[0], B[0], per, partials[0]);
    } else {
      allow_lds(k_gram<TGRAD_CBF16>, lds);
      k_gram<TGRAD_CBF16><<<grid, block, lds, s>>>(g, mask, A[0], In[0], B[0], per, partials[0]);
    }
    return;
  }
  GramJobs jobs;
  gram_line(njobs, A, In, B, groups, &jobs);
  size_t lds = 0;
  for (int i = 0; i < njobs; ++i) {
    GramJob& jb = jobs.job[i];
    jb.x = g;
    jb.mask = mask;
    jb.partials = partials[i];
    jb.magicB = B[i] <= 1 ? 0u : (uint32_t)((0x100000000ull + (uint64_t)B[i] - 1) / (uint64_t)B[i]);
    const size_t need = (size_t)4 * gram_plane(jb.rt) * sizeof(double);
    lds = need > lds ? need : lds;
  }
  const dim3 grid((unsigned)groups), block(kGram128Threads);
  if (dtype == TGRAD_C64) {
    allow_lds(k_gram128<TGRAD_C64>, lds);
    k_gram128<TGRAD_C64><<<grid, block, lds, s>>>(jobs);
  } else {
    allow_lds(k_gram128<TGRAD_CBF16>, lds);
    k_gram128<TGRAD_CBF16><<<grid, block, lds, s>>>(jobs);
  }
}

void launch_gram_reduce(hipStream_t s, int njobs, const int* In, const int* nchunks, double* const* partials,
                        double* const* gram) {
  ReduceJobs jobs;
  int64_t most = 1;
  for (int i = 0; i < njobs; ++i) {
    jobs.partials[i] = partials[i];
    jobs.gram[i] = gram[i];
    jobs.In[i] = In[i];
    jobs.nchunks[i] = nchunks[i];
    const int64_t n2 = (int64_t)In[i] * In[i];
    most = n2 > most ? n2 : most;
  }
  k_gram_reduce<<<dim3((unsigned)((most + kReduceElems - 1) / kReduceElems), (unsigned)njobs), dim3(256), 0, s>>>(jobs);
}

void launch_eig_batch(hipStream_t s, int njobs, const double* const* gram, double* const* work_a,
                      double* const* work_v, const int* In, const int* r, float* const* U, int* const* status,
                      int max_sweeps) {
  // max_sweeps == 0: the tridiagonal path first, Jacobi (full sweep budget) where it declines;
  // 1 .. kEigMaxSweeps: Jacobi with that budget for every solve
  const int use_fast = max_sweeps <= 0 ? 1 : 0;
  if (max_sweeps <= 0 || max_sweeps > kEigMaxSweeps) max_sweeps = kEigMaxSweeps;   // the log is sized for kEigMaxSweeps
  if (njobs <= 0) return;
  EigJobs small, large;                          // n <= 128: work matrix in LDS; larger: in memory
  int nsmall = 0, nlarge = 0, nmax = 0;
  for (int i = 0; i < njobs; ++i) {
    EigJob jb;
    jb.gram = gram[i];
    jb.A = work_a[i];
    jb.V = work_v[i];
    jb.U = U[i];
    jb.status = status[i];
    jb.n = In[i];
    jb.r = r[i];
    jb.max_sweeps = max_sweeps;
    jb.use_fast = In[i] <= kEigTriMaxN ? use_fast : 0;
    if (In[i] <= kEigTriMaxN) {
      small.job[nsmall++] = jb;
      if (In[i] > nmax) nmax = In[i];
    } else {
      large.job[nlarge++] = jb;
    }
  }
  if (nsmall > 0) {
    const size_t lds = (size_t)nmax * (nmax + 1) / 2 * sizeof(double2);
    static bool attr_set = false;
    if (!attr_set) {
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_eig_tri), hipFuncAttributeMaxDynamicSharedMemorySize,
                                kEigTriMaxN * (kEigTriMaxN + 1) / 2 * (int)sizeof(double2));
      attr_set = true;
    }
    if (use_fast) {
      int rmax = 1;
      for (int i = 0; i < nsmall; ++i) rmax = small.job[i].r > rmax ? small.job[i].r : rmax;
      const dim3 grid((unsigned)nsmall);
      if (nmax <= 64) k_trid<1><<<grid, dim3(256), 0, s>>>(small);
      else k_trid<2><<<grid, dim3(512), 0, s>>>(small);
      k_trid_vec<<<dim3((unsigned)rmax, (unsigned)nsmall), dim3(64), 0, s>>>(small);
    }
    k_eig_tri<<<dim3((unsigned)nsmall), dim3(kEigThreads), lds, s>>>(small);
    k_eig_apply<<<dim3((unsigned)nmax, (unsigned)nsmall), dim3(64), 0, s>>>(small);
    k_eig_finish<<<dim3((unsigned)nsmall), dim3(kEigThreads), 0, s>>>(small);
  }
  if (nlarge > 0) k_eig<<<dim3((unsigned)nlarge), dim3(kEigThreads), 0, s>>>(large);
}

void launch_identity_factor(hipStream_t s, float* U, int n) {
  k_identity_factor<<<dim3((unsigned)((n * n + 255) / 256)), dim3(256), 0, s>>>(
      reinterpret_cast<float2*>(U), n);
}

}  // namespace tgrad
