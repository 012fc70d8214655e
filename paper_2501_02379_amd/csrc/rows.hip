// First and last kernel of a step where modes N-1 and N are not done together (ends.hip does that for r_N <= 16 and
// r_(N-1) <= 32): the last mode alone, for rows of up to 72 elements and ranks up to 32, on split bf16 operands (device_common.h).
//   k_rows         g_S <- G[Omega];  out[row, m] = sum_i conj(U[i, m]) (G - Sparse(G, Omega))[row, i]
//   k_rows_update  W <- (1 - lr wd) W - lr (alpha z x_N U + lambda scatter(AdamUpdate(g_S)))
//
// A wavefront takes units of 16 rows (a tile of the matrix instructions), whatever their place in a slab, private to it from the
// first load to the last store; the support's offsets are those of 32 rows (k_tile_offsets), so both halves of 32 rows look through
// the same entries and each takes its own.  Coefficients of the mode lie in LDS in operand order, shared by the workgroup.
// The 32 x 32 kernels on float32 instructions (contract_mfma.hip), which have the longer rows, take units of 32 rows - two or three
// rounds of them for the wavefronts of a layer of a few million numbers - with 17 KB of LDS each and pad a rank of 18 to 32.
// Whole steps, us, with those / with these: 43x43x74x38, r 21,21,36,18 129 / 95, 24x24x128x65, r 8,8,40,32 128 / 92, 64x64x64x64,
// r 20,20,20,20 221 / 141, in bf16 50x50x64x64, r 10,10,20,32 152 / 93 (rows_kernel_pays and rows_update_pays have the kernels
// alone).  Relative error against 64 bits, those / these: k_rows with rows of 4, 16 and 72 elements 5.5e-8 / 3.9e-8, 1.0e-7 / 4.5e-8 and
// 2.2e-7 / 7.3e-8; k_rows_update with ranks 4, 16, 20 and 32 5.4e-8 / 4.3e-8, 1.0e-7 / 4.4e-8, 1.15e-7 / 1.12e-7 and 1.44e-7 / 9.6e-8.
//
// Lanes: g = lane / 16, c = lane % 16; slot 2 j + p of lane (c, g) is part p of element 16 quad + 4 j + g of row or column c;
// register r of a result is row 4 g + r, column c; real columns are (m, p) = (re, im) parts interleaved.
#include <type_traits>

#include "device_common.h"
#include "end_common.h"
#include "launch_util.h"

namespace tgrad {

namespace {

constexpr int kUnit = 16;                        // rows of a unit
constexpr int kRowsMaxWaves = 8;
constexpr int kRowsMaxExtent = 72;               // of the last mode: 9 pieces of 16 bytes per lane
constexpr int kRowsMaxRank = 32;

// Pieces of two complex elements (k_rows; complex64 W) per lane that cover a unit of rows of K elements: K / 8, in classes
int piece_class(int K) { return K <= 24 ? 3 : K <= 40 ? 5 : K <= 56 ? 7 : 9; }

// dwords of LDS per wavefront; an element takes ES of them (2, or 1 in bf16).  Rows of an even K are padded by one element, so that
// neighbouring rows do not share banks; what a commit writes past the unit and what the last row's quads read past its end
// lies inside.
__host__ __device__ inline int rows_slice(int ES, int K, int TB) {
  const int pad = (K & 1) ? 0 : 1, committed = TB * 64 * 2;
  const int a = committed + pad * (committed / K + 1), b = kUnit * (K + pad);
  return (ES * ((a > b ? a : b) + 16 * ((K + 15) / 16) + 4) + 3) & ~3;
}

// Coefficients into LDS, [item][h, m, l][lane], an item per operand of 16 elements and 16 columns: value(item, j) is what slot
// pair j of the lane's column meets.  Four items of a wavefront are requested together.
template <typename Value>
__device__ __forceinline__ void stage_coefs(u32v4* dst, int items, int wave, int W, int lane, Value value) {
  constexpr int kItems = 4;
  for (int i0 = wave; i0 < items; i0 += kItems * W) {
    float2 f[kItems][4];
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
      const int i = i0 + u * W < items ? i0 + u * W : i0;
#pragma unroll
      for (int j = 0; j < 4; ++j) f[u][j] = value(i, j);
    }
#pragma unroll
    for (int u = 0; u < kItems; ++u)
      if (i0 + u * W < items) {
        Split8 c;
#pragma unroll
        for (int j = 0; j < 4; ++j) split_at(c, j, f[u][j]);
        u32v4* p = dst + (i0 + u * W) * 192 + lane;
        p[0] = c.h;
        p[64] = c.m;
        p[128] = c.l;
      }
  }
}

struct RowsArgs {
  const void* g;
  const int32_t* omega;
  const uint32_t* tile_start;   // support entries below every 32 rows
  float2* gs;
  const float2* U;              // (K, M)
  float* out;                   // (rows, M) complex
  int K, M, nrows, nunits;
  uint32_t magicK;
};

// NC: tiles of 16 real columns (2 M)
template <int DT, int TB, int NC>
__global__ __launch_bounds__(64 * kRowsMaxWaves, 2) void k_rows(RowsArgs a) {
  typedef typename BufPair<DT>::type Raw;
  constexpr int kPiece = (int)sizeof(Raw), kElem = kPiece / 2, ES = kElem / 4;
  extern __shared__ float smem[];
  const int K = a.K, M = a.M, QN = (K + 15) >> 4;
  const int pad = (K & 1) ? 0 : 1, stride = ES * (K + pad), slice = rows_slice(ES, K, TB);
  const int W = (int)blockDim.x >> 6;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  float* sX = smem + wave * slice;
  u32v4* sC = reinterpret_cast<u32v4*>(smem + W * slice);                // conj(U) in operand order [quad][nc]
  const int nw = (int)gridDim.x * W;
  int unit = (int)blockIdx.x * W + wave;
  Raw raw[2][TB];                                                        // the units in flight
  u32x2 lone[2];                                                         // last element of a unit with an odd count
  auto elements = [&](int u) -> int {
    const int left = a.nrows - u * kUnit;
    return u < a.nunits ? (left < kUnit ? left : kUnit) * K : 0;
  };
  auto issue_unit = [&](Raw* to, u32x2& last, int u) {                   // (no unit: empty descriptors)
    const int n = elements(u), bytes = (n >> 1) * kPiece;
    const char* base = reinterpret_cast<const char*>(a.g) + (n ? (uint64_t)(uint32_t)u * (uint32_t)(kUnit * K) * kElem : 0ull);
#pragma unroll
    for (int k = 0; k < (TB + 3) / 4; ++k) {                             // a descriptor per 4 pieces: immediates reach 4 KB
      const int left = bytes - k * 4 * 64 * kPiece;
      const __amdgpu_buffer_rsrc_t r = raw_buffer(base + k * 4 * 64 * kPiece, (uint32_t)(left > 0 ? left : 0));
#pragma unroll
      for (int i = 4 * k; i < 4 * k + 4 && i < TB; ++i) to[i] = BufPair<DT>::load(r, lane * kPiece + (i - 4 * k) * 64 * kPiece);
    }
    const __amdgpu_buffer_rsrc_t rl = raw_buffer(base + bytes, (n & 1) ? kElem : 0);
    if constexpr (DT == TGRAD_C64) last = __builtin_amdgcn_raw_buffer_load_b64(rl, lane * kElem, 0, 2);
    else last.x = __builtin_amdgcn_raw_buffer_load_b32(rl, lane * kElem, 0, 2);
  };
  int32_t my_om = 0;
  auto issue_support = [&](uint32_t j0, uint32_t j1) {                   // the first 64 entries of the unit's 32 rows
    const uint32_t n = j1 - j0;
    my_om = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(raw_buffer(a.omega + j0, (n < 64u ? n : 64u) * 4u), lane * 4, 0, 0);
  };
  const uint32_t vzero = (uint32_t)opaque_zero();
  auto range_of = [&](int u, uint32_t& j0, uint32_t& j1) {               // per-lane loads, made scalar when used
    const uint32_t* ts = a.tile_start + (u < a.nunits ? u >> 1 : 0);
    j0 = ts[vzero];
    j1 = ts[vzero + 1];
  };
  // ---- prologue: the first units, then the operands go in flight ----
#pragma unroll
  for (int d = 0; d < 2; ++d) lone[d] = (u32x2){0u, 0u};
  issue_unit(raw[0], lone[0], unit);
  uint32_t cj0v, cj1v, nj0v, nj1v;
  range_of(unit, cj0v, cj1v);
  range_of(unit + nw, nj0v, nj1v);
  const FactorRef fU = factor_ref(a.U, (int64_t)K * M);
  stage_coefs(sC, QN * NC, wave, W, lane, [&](int i, int j) -> float2 {
    const int q = i / NC, nc = i - q * NC, k = 16 * q + 4 * j + grp, m = (16 * nc + col) >> 1;
    const float2 u = factor_entry(fU, k, m, M, k < K && m < M);
    return column_coef(make_float2(u.x, -u.y), col & 1);
  });
  for (int e = lane; e < slice; e += 64) sX[e] = 0.f;                    // pads stay finite
  int wofs[TB];                                                          // where the lane's pieces lie in the slice
#pragma unroll
  for (int i = 0; i < TB; ++i) {
    const int pi = lane + 64 * i;
    wofs[i] = ES * (2 * pi + (pad ? (int)div_magic(2u * (uint32_t)pi, a.magicK) : 0));
  }
  uint32_t cj0 = __builtin_amdgcn_readfirstlane(cj0v), cj1 = __builtin_amdgcn_readfirstlane(cj1v);
  if (unit >= a.nunits) cj1 = cj0;
  issue_support(cj0, cj1);
  issue_unit(raw[1], lone[1], unit + nw);
  __syncthreads();                                                       // the only workgroup barrier

  int ofs[NC];                                                           // columns past 2 M: dropped by the range check
#pragma unroll
  for (int nc = 0; nc < NC; ++nc)
    ofs[nc] = 16 * nc + col < 2 * M ? 4 * grp * (2 * M * 4) + (16 * nc + col) * 4 : 0x40000000;
  auto process = [&](auto set) {
    constexpr int D = decltype(set)::value;
    const int n_e = elements(unit);
    const uint32_t e_base = (uint32_t)unit * (uint32_t)(kUnit * K);      // I < 2^31
    wave_sync();                                                         // the previous unit's LDS reads are done
    asm volatile("" : "+v"(my_om), "+v"(lone[D]));
#pragma unroll
    for (int i = 0; i < TB; ++i) asm volatile("" : "+v"(raw[D][i]));     // one wait for the whole batch
#pragma unroll
    for (int i = 0; i < TB; ++i) {
      if constexpr (DT == TGRAD_C64) {
        float2* d = reinterpret_cast<float2*>(sX + wofs[i]);
        d[0] = make_float2(__uint_as_float(raw[D][i].x), __uint_as_float(raw[D][i].y));
        d[1] = make_float2(__uint_as_float(raw[D][i].z), __uint_as_float(raw[D][i].w));
      } else {
        uint32_t* d = reinterpret_cast<uint32_t*>(sX + wofs[i]);
        d[0] = raw[D][i].x;
        d[1] = raw[D][i].y;
      }
    }
    if (n_e & 1) {                                                       // (K is odd: no padding in the slice)
      wave_sync();
      if (lane == 0) {
        float* d = sX + ES * (n_e - 1);
        if constexpr (DT == TGRAD_C64) *reinterpret_cast<float2*>(d) = make_float2(__uint_as_float(lone[D].x), __uint_as_float(lone[D].y));
        else *reinterpret_cast<uint32_t*>(d) = lone[D].x;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // the next requests, in the order in which they are waited for (loads retire in order)
    const int32_t cur_om = my_om;
    const uint32_t nj0 = __builtin_amdgcn_readfirstlane(nj0v);
    const uint32_t nj1 = unit + nw < a.nunits ? (uint32_t)__builtin_amdgcn_readfirstlane(nj1v) : nj0;
    issue_support(nj0, nj1);
    range_of(unit + 2 * nw, nj0v, nj1v);
    issue_unit(raw[D], lone[D], unit + 2 * nw);
    wave_sync();
    {                                                                    // Sparse(G, Omega): hand the values over, then remove them
      auto take = [&](uint32_t j, int32_t oj) {
        const uint32_t e = (uint32_t)oj - e_base;
        if (e >= (uint32_t)n_e) return;                                  // of the other half of the 32 rows
        float* p = sX + ES * (e + (pad ? div_magic(e, a.magicK) : 0u));
        a.gs[cj0 + j] = load_elem<DT>(p, 0);
        if constexpr (DT == TGRAD_C64) *reinterpret_cast<float2*>(p) = make_float2(0.f, 0.f);
        else *reinterpret_cast<uint32_t*>(p) = 0u;
      };
      const uint32_t cnt = cj1 - cj0;
      if ((uint32_t)lane < cnt) take((uint32_t)lane, cur_om);
      if (cnt > 64u)
        for (uint32_t j = 64u + lane; j < cnt; j += 64) take(j, a.omega[cj0 + j]);
    }
    wave_sync();
    v4f y[NC], yl[NC];                                                   // the small terms have sums of their own
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) y[nc] = yl[nc] = (v4f){0.f, 0.f, 0.f, 0.f};
    const float* xa = sX + col * stride + ES * grp;
    const u32v4* cp = sC + lane;
    for (int q = 0; q < QN; ++q, xa += ES * 16, cp += NC * 192) {
      Split8 x;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float* p = xa + ES * 4 * j;
        if constexpr (DT == TGRAD_C64) split_at(x, j, *reinterpret_cast<const float2*>(p));
        else x.h[j] = *reinterpret_cast<const uint32_t*>(p);
      }
      u32v4 c[NC];
      auto operand = [&](int part) {
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) c[nc] = cp[nc * 192 + part * 64];
      };
      auto product = [&](const u32v4& xv, v4f* to) {
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) to[nc] = mfma_bf(xv, c[nc], to[nc]);
      };
      operand(2);
      product(x.h, yl);
      operand(1);
      if constexpr (DT == TGRAD_C64) product(x.m, yl);                   // (bf16 is its own first part)
      product(x.h, yl);
      operand(0);
      if constexpr (DT == TGRAD_C64) {
        product(x.l, yl);
        product(x.m, yl);
      }
      product(x.h, y);
    }
    const int row_bytes = 2 * M * 4, rows = a.nrows - unit * kUnit < kUnit ? a.nrows - unit * kUnit : kUnit;
    const char* ob = reinterpret_cast<const char*>(a.out) + (int64_t)unit * kUnit * row_bytes;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int left = (rows - r) * row_bytes;
      const __amdgpu_buffer_rsrc_t ro = raw_buffer(ob + r * row_bytes, (uint32_t)(left > 0 ? left : 0));
#pragma unroll
      for (int nc = 0; nc < NC; ++nc)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y[nc][r] + yl[nc][r]), ro, ofs[nc], 0, 0);
    }
    unit += nw;
    cj0 = nj0;
    cj1 = nj1;
  };
  while (unit < a.nunits) {
    process(std::integral_constant<int, 0>());
    if (unit >= a.nunits) break;
    process(std::integral_constant<int, 1>());
  }
}

struct RowsUpdateArgs {
  const float2* z;              // (rows, K) complex
  const float2* U;              // (M, K)
  void* w;
  int K, M, nrows, nunits;
  float decay, c_alpha;
};

// T: classes of M (pieces of complex64 W, column tiles of 16); Q: quads of K
template <int WDT, int T, int Q>
__global__ __launch_bounds__(64 * kRowsMaxWaves, 2) void k_rows_update(RowsUpdateArgs a, SparseAdam sp) {
  typedef WStore<WDT> WS;
  typedef typename WS::raw wraw;
  constexpr int kPre = WS::kElems == 2 ? T : (T + 1) / 2, kElem = 16 / WS::kElems;   // (bytes of an element of W)
  extern __shared__ float smem[];
  const int K = a.K, M = a.M, N2 = 2 * M, NT = (N2 + 15) >> 4;
  const int slice = (kUnit * N2 + 3) & ~3;
  const int W = (int)blockDim.x >> 6;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  float* sD = smem + wave * slice;
  u32v4* sC = reinterpret_cast<u32v4*>(smem + W * slice);                // c_alpha U in operand order [column tile][quad]
  const int nw = (int)gridDim.x * W;
  int unit = (int)blockIdx.x * W + wave;
  wraw wpre[2][kPre];                                                    // the units in flight
  uint32_t wl0[2], wl1[2];                                               // elements past the last whole piece of a unit
  auto elements = [&](int u) -> int {
    const int left = a.nrows - u * kUnit;
    return u < a.nunits ? (left < kUnit ? left : kUnit) * M : 0;
  };
  auto address = [&](int u) -> char* { return reinterpret_cast<char*>(a.w) + (uint64_t)(uint32_t)u * (uint32_t)(kUnit * M) * kElem; };
  auto issue_w = [&](wraw* to, uint32_t& l0, uint32_t& l1, int u) {      // (no unit: empty descriptors)
    const int n = elements(u), n4 = n / WS::kElems;
    const char* base = n ? address(u) : reinterpret_cast<const char*>(a.w);
#pragma unroll
    for (int k = 0; k < (kPre + 3) / 4; ++k) {                           // a descriptor per 4 pieces: immediates reach 4 KB
      const int left = n4 * 16 - k * 4096;
      const __amdgpu_buffer_rsrc_t r = raw_buffer(base + k * 4096, (uint32_t)(left > 0 ? left : 0));
#pragma unroll
      for (int i = 4 * k; i < 4 * k + 4 && i < kPre; ++i) buffer_piece_load(to[i], r, lane * 16 + (i - 4 * k) * 1024);
    }
    const __amdgpu_buffer_rsrc_t rl = raw_buffer(base + n4 * 16, (uint32_t)((n - n4 * WS::kElems) * kElem));
    if constexpr (WDT == TGRAD_C64) {
      const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rl, lane * kElem, 0, 0);
      l0 = v.x;
      l1 = v.y;
    } else {
      l0 = __builtin_amdgcn_raw_buffer_load_b32(rl, lane * kElem, 0, 0);
    }
  };
  int32_t my_om = 0;
  u32x2 my_g = {0u, 0u}, my_m = {0u, 0u};
  uint32_t my_v = 0;
  auto issue_sparse = [&](uint32_t j0, uint32_t j1) {                    // the first 64 entries of the unit's 32 rows
    const uint32_t n = j1 - j0 < 64u ? j1 - j0 : 64u;
    my_om = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(raw_buffer(sp.omega + j0, n * 4u), lane * 4, 0, 0);
    my_g = __builtin_amdgcn_raw_buffer_load_b64(raw_buffer(sp.gs + j0, n * 8u), lane * 8, 0, 0);
    my_m = __builtin_amdgcn_raw_buffer_load_b64(raw_buffer(sp.ms + j0, n * 8u), lane * 8, 0, 0);
    my_v = __builtin_amdgcn_raw_buffer_load_b32(raw_buffer(sp.vs + j0, n * 4u), lane * 4, 0, 0);
  };
  float2 z[Q][4];
  auto fetch_z = [&](int u) {                                            // rows past the end are not streamed, elements meet zeros
    const int row = u * kUnit + col;
    const float2* zr = a.z + (int64_t)(row < a.nrows ? row : a.nrows - 1) * K;
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = 16 * q + 4 * j + grp;
        z[q][j] = zr[k < K ? k : K - 1];
      }
  };
  const uint32_t vzero = (uint32_t)opaque_zero();
  auto range_of = [&](int u, uint32_t& j0, uint32_t& j1) {
    const uint32_t* ts = sp.tile_start + (u < a.nunits ? u >> 1 : 0);
    j0 = ts[vzero];
    j1 = ts[vzero + 1];
  };
  // ---- prologue: the first units of W, their operands and the coefficients go in flight ----
#pragma unroll
  for (int d = 0; d < 2; ++d) wl0[d] = wl1[d] = 0;
  issue_w(wpre[0], wl0[0], wl1[0], unit);
  uint32_t cj0v, cj1v, nj0v, nj1v;
  range_of(unit, cj0v, cj1v);
  range_of(unit + nw, nj0v, nj1v);
  fetch_z(unit < a.nunits ? unit : 0);
  const FactorRef fU = factor_ref(a.U, (int64_t)M * K);
  stage_coefs(sC, NT * Q, wave, W, lane, [&](int i, int j) -> float2 {
    const int q = i % Q, m = (16 * (i / Q) + col) >> 1, k = 16 * q + 4 * j + grp;
    const float2 u = factor_entry(fU, m, k, K, k < K && m < M);
    return column_coef(make_float2(a.c_alpha * u.x, a.c_alpha * u.y), col & 1);
  });
  uint32_t cj0 = __builtin_amdgcn_readfirstlane(cj0v), cj1 = __builtin_amdgcn_readfirstlane(cj1v);
  if (unit >= a.nunits) cj1 = cj0;
  issue_sparse(cj0, cj1);
  issue_w(wpre[1], wl0[1], wl1[1], unit + nw);
  __syncthreads();                                                       // the only workgroup barrier
  auto process = [&](auto set) {
    constexpr int D = decltype(set)::value;
    const uint32_t w_base = (uint32_t)unit * (uint32_t)(kUnit * M);
    const int n_w = elements(unit), n4 = n_w / WS::kElems;
    Split8 za[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) split_at(za[q], j, z[q][j]);
    fetch_z(unit + nw < a.nunits ? unit + nw : unit);
    wave_sync();                                                         // the previous unit's LDS reads are done
    float* sR = sD + 4 * grp * N2 + col;
#pragma unroll
    for (int i0 = 0; i0 < T; i0 += 2) {
      if (i0 < NT) {                                                     // (wave-uniform)
        constexpr int kTwo = 2;
        v4f o[kTwo] = {(v4f){0.f, 0.f, 0.f, 0.f}, (v4f){0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          Split8 b[kTwo];
#pragma unroll
          for (int u = 0; u < kTwo; ++u) {
            const u32v4* p = sC + ((i0 + u < NT ? i0 + u : i0) * Q + q) * 192 + lane;
            b[u] = Split8{p[0], p[64], p[128]};
          }
          mfma_split<kTwo>(o, za[q], b);
        }
#pragma unroll
        for (int u = 0; u < kTwo; ++u)
          if (16 * (i0 + u) + col < N2) {
#pragma unroll
            for (int r = 0; r < 4; ++r) sR[r * N2 + 16 * (i0 + u)] = o[u][r];
          }
      }
    }
    wave_sync();
    // ---- AdamUpdate on the sparse values that live in this unit; add lambda N_S into it ----
    {
      const uint32_t cnt = cj1 - cj0;
      auto mine = [&](int32_t oj) -> bool { return (uint32_t)oj - w_base < (uint32_t)n_w; };
      if ((uint32_t)lane < cnt && mine(my_om))
        sparse_adam_entry(sp, cj0 + lane, my_om, make_float2(__uint_as_float(my_g.x), __uint_as_float(my_g.y)),
                          make_float2(__uint_as_float(my_m.x), __uint_as_float(my_m.y)), __uint_as_float(my_v),
                          (int64_t)w_base, sD);
      if (cnt > 64u)                                                     // more than 64 entries in 32 rows
        for (uint32_t j = cj0 + 64u + lane; j < cj1; j += 64) {
          const int32_t oj = sp.omega[j];
          if (mine(oj)) sparse_adam_entry(sp, j, oj, sp.gs[j], sp.ms[j], sp.vs[j], (int64_t)w_base, sD);
        }
    }
    wave_sync();
    // ---- stream the unit into W ----
    char* w_unit = address(unit);
#pragma unroll
    for (int i = 0; i < kPre; ++i) claim_raw(wpre[D][i]);
#pragma unroll
    for (int k = 0; k < (kPre + 3) / 4; ++k) {
      const int left = n4 * 16 - k * 4096;
      const __amdgpu_buffer_rsrc_t r = raw_buffer(w_unit + k * 4096, (uint32_t)(left > 0 ? left : 0));
#pragma unroll
      for (int i = 4 * k; i < 4 * k + 4 && i < kPre; ++i) {
        const int q = lane + i * 64;                                     // (the LDS read stays inside the slice)
        buffer_piece_store(WS::apply(wpre[D][i], sD, q < n4 ? q : 0, a.decay), r, lane * 16 + (i - 4 * k) * 1024);
      }
    }
    {                                                                    // elements past the last whole piece
      const int e = n4 * WS::kElems + lane;
      if (e < n_w) {
        if constexpr (WDT == TGRAD_C64)
          *reinterpret_cast<float2*>(w_unit + (int64_t)e * kElem) =
              make_float2(a.decay * __uint_as_float(wl0[D]) + sD[2 * e], a.decay * __uint_as_float(wl1[D]) + sD[2 * e + 1]);
        else
          *reinterpret_cast<uint32_t*>(w_unit + (int64_t)e * kElem) =
              WStore<TGRAD_CBF16>::one(wl0[D], sD[2 * e], sD[2 * e + 1], a.decay);
      }
    }
    // ---- the next units go in flight: the support first, which the next one waits for (loads retire in order) ----
    cj0 = __builtin_amdgcn_readfirstlane(nj0v);
    cj1 = unit + nw < a.nunits ? (uint32_t)__builtin_amdgcn_readfirstlane(nj1v) : cj0;
    issue_sparse(cj0, cj1);
    range_of(unit + 2 * nw, nj0v, nj1v);
    issue_w(wpre[D], wl0[D], wl1[D], unit + 2 * nw);
    unit += nw;
  };
  while (unit < a.nunits) {
    process(std::integral_constant<int, 0>());
    if (unit >= a.nunits) break;
    process(std::integral_constant<int, 1>());
  }
}

// ---- host side ----------------------------------------------------------------------------------

size_t rows_lds(int W, int es, int K, int M) {
  return (size_t)W * rows_slice(es, K, piece_class(K)) * 4 + (size_t)((K + 15) / 16) * ((2 * M + 15) / 16) * 3072;
}
size_t rows_update_lds(int W, int M, int K) {
  return (size_t)W * ((kUnit * 2 * M + 3) & ~3) * 4 + (size_t)((2 * M + 15) / 16) * ((K + 15) / 16) * 3072;
}

// Wavefronts per workgroup: 4 where two such workgroups fit a compute unit, or 8 that fit one
int rows_waves(size_t lds4, size_t lds8) { return lds4 <= kLdsLimit / 2 ? 4 : lds8 <= kLdsLimit ? 8 : 4; }

template <typename Kern>
unsigned rows_grid(Kern kern, int W, size_t lds, int64_t units) {
  const int64_t groups = (units + W - 1) / W, cap = (int64_t)compute_units() * resident_blocks(kern, 64 * W, lds, 8);
  return (unsigned)(groups < cap ? groups : cap);
}

}  // namespace

// Extent K and rank r of the last mode.
static bool rows_kernel_fits(int K, int r) { return K >= 2 && K <= kRowsMaxExtent && r <= kRowsMaxRank; }

// k_rows takes nearly all of these from k_lproj; us, k_lproj / k_rows, rows x K, r: 12288x4, 1 4.6 / 4.2; 12288x33, 8 7.8 / 5.3; 229376x4, 1
// 9.7 / 9.0; 229376x33, 8 26 / 18; 400000x20, 5 29 / 20; 160000x65, 8 34 / 23; 640000x12, 10 34 / 32; 640000x65, 16 109 / 80; 640000x33, 17 86 / 58;
// 640000x72, 30 288 / 113.  Not rows of up to 6 elements where they are one to six units for each wavefront of the chip, half as many
// tiles for k_lproj (whole step: 65536x3 27.7 / 29.4, 98304x4 29.6 / 30.8, 65536x5 28.4 / 29.5, 76800x5 30.3 / 30.7, bf16 152047x3 36.8 /
// 38.0; a launch, 151872 rows of 2 to 6: 7.4 .. 8.7 / 8.0 .. 9.0, in bf16 7.2 .. 8.6 / 8.6 .. 9.8; but 204800x3 40.1 / 38.8 and launches
// of 375000 rows of 2 to 6 12.4 .. 15.8 / 12.2 .. 13.7).
bool rows_kernel_pays(int K, int r, int64_t rows) {
  return rows_kernel_fits(K, r) && (K > 6 || rows < 1024 * kUnit || rows >= 12288 * kUnit);
}

// k_rows_update leaves ranks up to 8 of many rows to k_lupdate, which has two matrix steps of four elements for them and half as
// many units to go around: 229376x4, r 1 7.9 / 12.6; 400000x12, r 3 18.2 / 24.0; 400000x20, r 5 27.4 / 30.0; 160000x65, r 8 34.0 / 34.7;
// but 640000x12, r 10 38.8 / 36.8; 640000x24, r 9 58 / 51; 640000x65, r 16 136 / 127; 640000x33, r 17 101 / 77; 640000x72, r 30 350 /
// 153; and with a wavefront for every unit 12288x24, r 6 5.8 / 4.8.  Ranks 1 and 2 stay there in any number (12288x4, r 1 4.3 /
// 3.9): what the six products of three parts leave out is more than two or four float32 multiply-adds round off (relative error
// 3.1e-8 / 4.4e-8 at 2 columns of rank 1, 3.9e-8 / 4.1e-8 at 4 of rank 2; from rank 3 on 4.7e-8 / 4.2e-8 and less).
bool rows_update_pays(int K, int r, int64_t rows) {
  return rows_kernel_fits(K, r) && (r > 8 || (r > 2 && rows < 1024 * kUnit));
}

void launch_rows(hipStream_t s, const void* g, int dtype, const int32_t* omega, const uint32_t* tile_start, float2* gs,
                 const float2* U, const Stage& st, float2* out) {
  const int K = st.K, M = st.M, es = dtype == TGRAD_C64 ? 2 : 1;
  const int64_t units = (st.A + kUnit - 1) / kUnit;
  if (st.A * M <= 0) return;
  const int full = rows_waves(rows_lds(4, es, K, M), rows_lds(8, es, K, M)), W = units >= 1024 ? full : 1;
  const size_t lds = rows_lds(W, es, K, M);
  const RowsArgs a{g, omega, tile_start, gs, U, reinterpret_cast<float*>(out), K, M, (int)st.A, (int)units, magic_for(K)};
  const int tb = piece_class(K), nc = (2 * M + 15) / 16;
#define TGRAD_ROWS(DT_, T_, C_)                                                                              \
  do {                                                                                                       \
    allow_lds(k_rows<DT_, T_, C_>, lds);                                                                     \
    k_rows<DT_, T_, C_><<<dim3(rows_grid(k_rows<DT_, T_, C_>, W, lds, units)), dim3(64 * W), lds, s>>>(a);   \
  } while (0)
#define TGRAD_ROWS_C(DT_, T_)                                                                                \
  do {                                                                                                       \
    if (nc == 1) TGRAD_ROWS(DT_, T_, 1); else if (nc == 2) TGRAD_ROWS(DT_, T_, 2);                           \
    else if (nc == 3) TGRAD_ROWS(DT_, T_, 3); else TGRAD_ROWS(DT_, T_, 4);                                   \
  } while (0)
#define TGRAD_ROWS_T(DT_)                                                                                    \
  do {                                                                                                       \
    if (tb == 3) TGRAD_ROWS_C(DT_, 3); else if (tb == 5) TGRAD_ROWS_C(DT_, 5);                               \
    else if (tb == 7) TGRAD_ROWS_C(DT_, 7); else TGRAD_ROWS_C(DT_, 9);                                       \
  } while (0)
  if (dtype == TGRAD_C64) TGRAD_ROWS_T(TGRAD_C64); else TGRAD_ROWS_T(TGRAD_CBF16);
#undef TGRAD_ROWS
#undef TGRAD_ROWS_C
#undef TGRAD_ROWS_T
}

void launch_rows_update(hipStream_t s, const float2* z, const float2* U, const Stage& st, void* w, int wdtype, float decay,
                        float c_alpha, const int32_t* omega, const uint32_t* tile_start, const float2* gs, float2* ms, float* vs,
                        float beta1, float beta2, double inv_c1, double inv_c2, float eps, float c_lambda) {
  const int K = st.K, M = st.M;
  const int64_t units = (st.A + kUnit - 1) / kUnit;
  if (st.A * M <= 0) return;
  const int full = rows_waves(rows_update_lds(4, M, K), rows_update_lds(8, M, K)), W = units >= 1024 ? full : 1;
  const size_t lds = rows_update_lds(W, M, K);
  const RowsUpdateArgs a{z, U, w, K, M, (int)st.A, (int)units, decay, c_alpha};
  const SparseAdam sp = sparse_adam(omega, tile_start, gs, ms, vs, beta1, beta2, inv_c1, inv_c2, eps, c_lambda, 0);
  const int t = piece_class(M);
#define TGRAD_RU(WD_, T_, Q_)                                                                                \
  do {                                                                                                       \
    allow_lds(k_rows_update<WD_, T_, Q_>, lds);                                                              \
    k_rows_update<WD_, T_, Q_><<<dim3(rows_grid(k_rows_update<WD_, T_, Q_>, W, lds, units)), dim3(64 * W), lds, s>>>(a, sp); \
  } while (0)
#define TGRAD_RU_Q(WD_, T_) do { if (K <= 16) TGRAD_RU(WD_, T_, 1); else TGRAD_RU(WD_, T_, 2); } while (0)
#define TGRAD_RU_T(WD_)                                                                                      \
  do {                                                                                                       \
    if (t == 3) TGRAD_RU_Q(WD_, 3); else if (t == 5) TGRAD_RU_Q(WD_, 5); else if (t == 7) TGRAD_RU_Q(WD_, 7); \
    else TGRAD_RU_Q(WD_, 9);                                                                                 \
  } while (0)
  if (wdtype == TGRAD_C64) TGRAD_RU_T(TGRAD_C64); else TGRAD_RU_T(TGRAD_CBF16);
#undef TGRAD_RU
#undef TGRAD_RU_Q
#undef TGRAD_RU_T
}

}  // namespace tgrad
