// First and last kernel of a step on 16 x 16 matrix-core tiles, for any extent of mode N-1:
//   k_head  g_S <- G[Omega];  out[slab, m2, m3] = sum_{i2, i3} conj(U2[i2, m2]) conj(U3[i3, m3]) (G - Sparse(G, Omega))[slab, i2, i3]
//           (or of G itself, in the two orders in which the low-rank part sees the full gradient: a gather kernel of its own
//           took 8 us at 64x64x64x32 with 5 % of the entries, whole step 89 -> 82)
//   k_tail  W <- (1 - lr wd) W - lr (alpha z x_(N-1) U2 x_N U3 + lambda scatter(AdamUpdate(g_S)))
// with modes N-1 (extent I2, rank M2 <= 32) and N (extent K, rank M <= 16) in one pass over G and one over W; a
// slab is the I2 x K block of one set of leading indices.  (contract_mfma.hip has the same two passes on 32 x 32
// tiles, for few slabs of ranks that fill them: wide_tiles_pay has the line.)
//
// Why 16 x 16: a rank is padded to the tile, so a last-mode rank of 4 or 8 - which most layers have - and a rank up to 16 of
// mode N-1 cost a half to a quarter of the matrix work of 32-wide tiles.  Why split bf16 operands (device_common.h): in
// float32 instructions both passes were bound by them where ranks fill the tiles or elements are bf16 (70 to 80 % of the
// kernel's cycles), now they take 15 to 35 %, and memory, or the instructions around a small tile, bounds the pass.
//
// Measured (rocprofv3, us; 32 x 32 tiles or separate kernels -> 16 x 16 in float32 -> split operands):
//   first pass 64x64x32x17 15.7 -> 9.9 -> 9, 32x32x32x32x17 (bf16) 84.5 -> 34.8 -> 24, 128x128x64x33 91.7 -> 56 -> 55 (5.0 TB/s;
//   its loads alone 52.6), bf16 87.7 -> 46 -> 35, r 32,16 102 (32 x 32) -> 73, 128x128x128x65 243 (32 x 32) -> 222;
//   last pass 128x128x64x33 112 -> 108 -> 105 (5.3 TB/s), bf16 weights 98 -> 66 -> 60, r 32,16 140 (32 x 32) -> 109,
//   90x77x45x23 10.6 + 26.8 -> 28 -> 26.5, 128x128x128x65 434 (32 x 32) -> 440, slabs shared 426.
//
// Lanes: g = lane / 16, c = lane % 16.  A[i = c][k = g], B[k = g][j = c], D register r: D[i = 4 g + r][j = c].
// Real columns are (m, p) = (re, im) parts interleaved: c = 2 m + p.
//
// Tiles of R rows of a slab (R = 32; 16 where rows are long: end_tile_rows) belong to one wavefront from the
// first load to the last store and are staged in LDS private to it, as in contract_mfma.hip.  A wavefront walks
// whole slabs where there are enough of them to occupy the chip; with fewer (SPLIT) the wavefronts of a
// workgroup share a slab (k_head: partial sums added through LDS in a fixed order), or take any tile (k_tail).
#include <type_traits>

#include "device_common.h"
#include "end_common.h"
#include "launch_util.h"

namespace tgrad {

namespace {

constexpr int kMaxWaves = 8;

// v of the neighbouring lane (c ^ 1): the other part of the same complex column
__device__ __forceinline__ float swap_parts(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
}

// ---- k_head -------------------------------------------------------------------------------------
// Stage 1  y[row, (m3, p)] = sum_i3 conj(U3) G: quads of 16 elements of a row on split bf16 operands (device_common.h; slot
//   2 j + p of lane (c, g) is part p of element 16 quad + 4 j + g), a remainder of up to four elements - half-spectrum modes
//   have one - as a float32 step.  G in bf16 is its own first part and needs no others: three products instead of six, and no
//   vector arithmetic to prepare them.
// Stage 2  sums over 32 rows of the slab at a time: register r of y is row 4 g + r of its 16, so the eight values of two
//   16-row halves are the slots of a B operand as they stand; conj(U2) comes split from the table in LDS.
// T4: steps of four elements of K (class of K); quads and remainder steps that do them.
constexpr int head_quads(int T4) { return T4 / 4 + (T4 % 4 >= 2 ? 1 : 0); }
constexpr int head_rest(int T4) { return T4 % 4 == 1 ? 1 : 0; }
constexpr int head_rows(int T4) { return T4 <= 9 ? 32 : 16; }            // rows per tile
constexpr int head_pieces(int T4) { return T4 <= 9 ? T4 : (T4 + 1) / 2; }   // pieces of two elements per lane that cover a tile
// dwords of LDS per wavefront; an element takes ES of them (2, or 1 in bf16).  Rows of an even K are padded by one element,
// so that neighbouring rows do not share banks; everything a commit writes and everything the steps past K read lies
// inside, and so do the partial sums of a shared slab.
__host__ __device__ constexpr int head_slice(int ES, int K, int T4) {
  const int pad = (K & 1) ? 0 : 1;
  const int committed = head_pieces(T4) * 64 * 2;                        // elements that a commit writes
  const int a = committed + pad * (committed / K + 1);
  const int b = head_rows(T4) * (K + pad);
  const int c = ES * ((a > b ? a : b) + 16 * head_quads(T4) + 4);        // + what the last row's steps read past its end
  return ((c > 1024 ? c : 1024) + 3) & ~3;                               // 1024: partial sums of two by two tiles
}
// Tiles in flight per wavefront.  What a compute unit has in flight decides what it streams (64-row slabs of 33 elements:
// loads alone 4.5 TB/s with 67 KB, 5.3 with 100 KB); registers hold more of it than LDS would.  k_head with one / two: 6400
// slabs of 100x36, r 16,8 51 / 48 us, 10000 of 64x65 66 / 64, 16384 of 128x65, r 32,16 239 / 237, of 64x33, r 16,8 56 / 56.
constexpr int head_ahead(int T4, int NC) { return T4 >= 9 && NC == 2 ? 2 : T4 >= 13 ? 2 : 1; }
// Coefficients of two column tiles and more than two operands' worth each way are kept in LDS (a tile reads them once) where a
// wavefront has many tiles (HEAD_MANY), others in registers: with one column tile and rows of 34 to 68 elements LDS was up to
// 23 % slower (16384 slabs of 80x34, r 20,6 95 / 88 us; 2511 of 113x38, r 31,8 38 / 31).
constexpr bool head_many_coefs(int T4, int NC) { return head_quads(T4) * NC > 2; }
constexpr bool head_coef_lds(int T4, int NC) { return NC == 2 && head_many_coefs(T4, NC); }
constexpr int kHeadItem = 6 * 64;         // u32v4 of the table per 32 rows and tile of M2: (Fr, Fi) x (h, m, l) x lane

struct HeadArgs {
  const void* g;
  const int32_t* omega;
  const uint32_t* tile_start;   // support entries below every tile of every slab
  float2* gs;
  const float2* U3;             // (K, M)
  const float2* U2;             // (I2, M2)
  int K, M, I2, M2, S, nslabs;  // S: tiles per slab
  int split;
  int keep;                     // 1: the support is handed over, but not removed
  uint32_t magicK;
  float* out;                   // (nslabs, M2, M) complex
};

// What a launch of a class with many coefficients (head_many_coefs) looks like; the others are HEAD_MANY (but see head_has_one).
// Staging the coefficients, a second tile in flight and the waits between an operand in LDS and its product are worth their
// while where a wavefront has many tiles.  Where it has one or two they were 1.0 to 1.7 us of 7 to 8 (head_mode has the lines).
//   HEAD_MANY  wavefronts that walk whole slabs, workgroups that stay for several shared slabs
//   HEAD_FEW   shared slabs, coefficients in registers, one tile in flight
//   HEAD_ONE   one tile per wavefront: all of its operands in registers, no table, no next tile
enum HeadMode { HEAD_MANY, HEAD_FEW, HEAD_ONE };

// NC: tiles of 16 real columns (2 M), NM: tiles of 16 rows (M2)
template <int DT, int T4, int NC, int NM, int MODE>
__global__ __launch_bounds__(64 * kMaxWaves, 2) void k_head(HeadArgs a) {
  typedef typename BufPair<DT>::type Raw;
  constexpr int R = head_rows(T4), TB = head_pieces(T4);
  constexpr int kPiece = (int)sizeof(Raw), kElem = kPiece / 2;           // bytes of two elements, of one
  constexpr int ES = kElem / 4;                                          // dwords of an element in LDS
  constexpr int QN = head_quads(T4), REST = head_rest(T4), kAhead = MODE == HEAD_MANY ? head_ahead(T4, NC) : 1;
  constexpr bool ONE = MODE == HEAD_ONE;
  extern __shared__ float smem[];
  const int K = a.K, M = a.M, I2 = a.I2, M2 = a.M2, S = a.S;
  const int pad = (K & 1) ? 0 : 1, stride = ES * (K + pad);
  const int slice = head_slice(ES, K, T4);
  const int W = (int)blockDim.x >> 6;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  float* sX = smem + wave * slice;
  u32v4* sT = reinterpret_cast<u32v4*>(smem + W * slice);                // conj(U2) in operand order [32 rows][nm]
  const bool split = a.split != 0, keep = a.keep != 0;
  const int nw = (int)gridDim.x * W;
  int slab = split ? (int)blockIdx.x : (int)blockIdx.x * W + wave, ts = split ? wave : 0;
  if (ts >= S) slab = a.nslabs;                                          // (a shared slab with fewer tiles than wavefronts)
  auto advance = [&](int& sl, int& t) {
    if (split) {
      t += W;
      if (t >= S) sl = a.nslabs;
    } else if (t + 1 < S) {
      t += 1;
    } else {
      t = 0;
      sl += nw;
    }
  };
  const uint32_t slab_elems = (uint32_t)(I2 * K);
  Raw raw[kAhead][TB];                                                   // the tiles in flight
  u32x2 lone[kAhead];                                                    // last element of a tile with an odd count
  int32_t my_om = 0;
  // the tile being fetched (scalar): address, bytes in whole pieces (0: no tile), elements
  const char* f_base = reinterpret_cast<const char*>(a.g);
  int f_bytes = 0, f_n = 0;
  auto set_fetch = [&](int sl, int t) {
    const bool ok = sl < a.nslabs;
    const int rows = I2 - t * R < R ? I2 - t * R : R;
    f_n = ok ? rows * K : 0;
    f_bytes = (f_n >> 1) * kPiece;
    f_base = reinterpret_cast<const char*>(a.g) +
             (ok ? ((uint64_t)(uint32_t)sl * slab_elems + (uint32_t)(t * R * K)) * (uint64_t)kElem : 0ull);
  };
  auto issue_piece = [&](Raw* to, int i) {
    const int k = i / 4, left = f_bytes - k * 4 * 64 * kPiece;           // a descriptor per 4 pieces: immediates reach 4 KB
    const __amdgpu_buffer_rsrc_t r = raw_buffer(f_base + k * 4 * 64 * kPiece, (uint32_t)(left > 0 ? left : 0));
    to[i] = BufPair<DT>::load(r, lane * kPiece + (i - 4 * k) * 64 * kPiece);
  };
  auto issue_lone = [&](u32x2& to) {
    const __amdgpu_buffer_rsrc_t r = raw_buffer(f_base + f_bytes, (f_n & 1) ? kElem : 0);
    if constexpr (DT == TGRAD_C64) {
      to = __builtin_amdgcn_raw_buffer_load_b64(r, lane * kElem, 0, 2);
    } else {
      to.x = __builtin_amdgcn_raw_buffer_load_b32(r, lane * kElem, 0, 2);
    }
  };
  auto issue_support = [&](uint32_t j0, uint32_t j1) {
    const uint32_t cnt = j1 - j0;
    const __amdgpu_buffer_rsrc_t ro = raw_buffer(a.omega + j0, (cnt < 64u ? cnt : 64u) * 4u);
    my_om = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(ro, lane * 4, 0, 0);
  };
  // ---- prologue: the first tiles, then the operands go in flight ----
  int s1 = slab, t1 = ts;                                                // the tile after this one, the one after that
  if (slab < a.nslabs) advance(s1, t1);
  int s2 = s1, t2 = t1;
  if (s1 < a.nslabs) advance(s2, t2);
  auto issue_tile = [&](Raw* to, u32x2& last, int sl, int t) {
    set_fetch(sl, t);
#pragma unroll
    for (int i = 0; i < TB; ++i) issue_piece(to, i);
    last = (u32x2){0u, 0u};
    issue_lone(last);
  };
  issue_tile(raw[0], lone[0], slab, ts);
  const uint32_t vzero = (uint32_t)opaque_zero();
  auto range_of = [&](int sl, int t, uint32_t& j0, uint32_t& j1) {       // per-lane loads, made scalar when used
    const uint32_t* tsb = a.tile_start + (sl < a.nslabs ? (int64_t)sl * S + t : 0);
    j0 = tsb[vzero];
    j1 = tsb[vzero + 1];
  };
  uint32_t cj0v, cj1v, nj0v, nj1v;
  range_of(slab, ts, cj0v, cj1v);
  if constexpr (!ONE) range_of(s1, t1, nj0v, nj1v);
  const FactorRef fU3 = factor_ref(a.U3, (int64_t)K * M), fU2 = factor_ref(a.U2, (int64_t)I2 * M2);
  constexpr bool kInLds = MODE == HEAD_MANY && head_coef_lds(T4, NC);
  Split8 cq[kInLds ? 1 : QN][NC];                                        // conj(U3)[16 q + 4 j + g][column]
  u32v4* sC = sT + ((I2 + 31) >> 5) * (NM * kHeadItem);
  float2 crest[NC];
  auto coef = [&](int k, int nc) -> float2 {
    const int m = (16 * nc + col) >> 1;
    const float2 u = factor_entry(fU3, k, m, M, k < K && m < M);
    return column_coef(make_float2(u.x, -u.y), col & 1);
  };
#pragma unroll
  for (int nc = 0; nc < NC; ++nc) {
    if constexpr (!kInLds && !ONE) {
#pragma unroll
      for (int q = 0; q < QN; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) split_at(cq[q][nc], j, coef(16 * q + 4 * j + grp, nc));
    }
    if constexpr (REST > 0) crest[nc] = coef(16 * QN + grp, nc);
  }
  const int items = ((I2 + 31) >> 5) * NM * 64;
  auto table_load = [&](int e, float2* u) {                              // (past the end: zeros)
    const int l = e & 63, nm = (e >> 6) % NM, q = (e >> 6) / NM;
    const int m2 = 16 * nm + (l & 15);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int i2 = 32 * q + 16 * (i >> 2) + 4 * (l >> 4) + (i & 3);
      u[i] = factor_entry(fU2, i2, m2, M2, i2 < I2 && m2 < M2);
    }
  };
  auto table_split = [&](const float2* u, Split8& fr, Split8& fi) {      // conj(U2): (Fr, Fi)
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      split_at(fr, d, make_float2(u[2 * d].x, u[2 * d + 1].x));
      split_at(fi, d, make_float2(-u[2 * d].y, -u[2 * d + 1].y));
    }
  };
  uint32_t cj0, cj1;
  auto first_support = [&]() {
    cj0 = __builtin_amdgcn_readfirstlane(cj0v);
    cj1 = slab < a.nslabs ? __builtin_amdgcn_readfirstlane(cj1v) : cj0;
    issue_support(cj0, cj1);
  };
  Split8 own_r[ONE ? NM : 1], own_i[ONE ? NM : 1];                       // (ONE) the table's rows of this wavefront's tile
  if constexpr (ONE) {
    float2 f[QN][NC][4], u[NM][8];
#pragma unroll
    for (int q = 0; q < QN; ++q)
#pragma unroll
      for (int nc = 0; nc < NC; ++nc)
#pragma unroll
        for (int j = 0; j < 4; ++j) f[q][nc][j] = coef(16 * q + 4 * j + grp, nc);
#pragma unroll
    for (int nm = 0; nm < NM; ++nm) table_load(((R == 32 ? ts : ts >> 1) * NM + nm) * 64 + lane, u[nm]);
    for (int e = lane; e < slice; e += 64) sX[e] = 0.f;                  // pads stay finite
    __builtin_amdgcn_sched_barrier(0);
    first_support();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < QN; ++q)
#pragma unroll
      for (int nc = 0; nc < NC; ++nc)
#pragma unroll
        for (int j = 0; j < 4; ++j) split_at(cq[q][nc], j, f[q][nc][j]);
#pragma unroll
    for (int nm = 0; nm < NM; ++nm) table_split(u[nm], own_r[nm], own_i[nm]);
  }
  float2 tu[8];
  if constexpr (kInLds) table_load(tid, tu);                             // in flight under the coefficients
  if constexpr (kInLds) {
    // [q][nc][h, m, l][lane]; a wavefront's next operands are requested together (a round trip each was 2 us of the 18 that
    // a step of 42x42x44 takes)
    constexpr int kItems = QN * NC < 4 ? QN * NC : 4;
    for (int i0 = wave; i0 < QN * NC; i0 += kItems * W) {
      float2 f[kItems][4];
#pragma unroll
      for (int u = 0; u < kItems; ++u) {
        const int i = i0 + u * W < QN * NC ? i0 + u * W : i0, q = i / NC, nc = i % NC;
#pragma unroll
        for (int j = 0; j < 4; ++j) f[u][j] = coef(16 * q + 4 * j + grp, nc);
      }
#pragma unroll
      for (int u = 0; u < kItems; ++u)
        if (i0 + u * W < QN * NC) {
          Split8 c;
#pragma unroll
          for (int j = 0; j < 4; ++j) split_at(c, j, f[u][j]);
          u32v4* p = sC + (i0 + u * W) * 192 + lane;
          p[0] = c.h;
          p[64] = c.m;
          p[128] = c.l;
        }
    }
  }
  if constexpr (!ONE) {
    for (int e = lane; e < slice; e += 64) sX[e] = 0.f;                  // pads stay finite
    for (int e = tid; e < items; e += (int)blockDim.x) {
      if (!kInLds || e != tid) table_load(e, tu);
      Split8 fr, fi;
      table_split(tu, fr, fi);
      u32v4* p = sT + (e >> 6) * kHeadItem + (e & 63);
      p[0] = fr.h; p[64] = fr.m; p[128] = fr.l;
      p[192] = fi.h; p[256] = fi.m; p[320] = fi.l;
    }
  }
  int wofs[TB];                                                          // where the lane's pieces lie in the slice
#pragma unroll
  for (int i = 0; i < TB; ++i) {
    const int pi = lane + 64 * i;
    wofs[i] = ES * (2 * pi + (pad ? (int)div_magic(2u * (uint32_t)pi, a.magicK) : 0));
  }
  if constexpr (!ONE) first_support();
  if constexpr (kAhead > 1) issue_tile(raw[kAhead - 1], lone[kAhead - 1], s1, t1);   // (the loop's order of requests)
  if constexpr (!ONE) __syncthreads();                                   // (the only barrier unless the slab is shared)
  if (!split && slab >= a.nslabs) return;

  // second-stage sums, unswapped: da = sum fr y, db = sum fi y (db of the other part is exchanged once per slab)
  v4f da[NM][NC], db[NM][NC];
  auto clear = [&]() {
#pragma unroll
    for (int nm = 0; nm < NM; ++nm)
#pragma unroll
      for (int nc = 0; nc < NC; ++nc) da[nm][nc] = db[nm][nc] = (v4f){0.f, 0.f, 0.f, 0.f};
  };
  auto value = [&](int nm, int nc, int r) -> float {                     // re: a_re - b_im, im: a_im + b_re
    const float s = swap_parts(db[nm][nc][r]);
    return (col & 1) ? da[nm][nc][r] + s : da[nm][nc][r] - s;
  };
  // out[sl, m2, column] through a descriptor that ends with the slab: rows past M2 are dropped by the range check,
  // columns past 2 M by an offset beyond it
  const int row_bytes = 2 * M * 4;
  int ofs[NC];
#pragma unroll
  for (int nc = 0; nc < NC; ++nc)
    ofs[nc] = 16 * nc + col < 2 * M ? 4 * grp * row_bytes + (16 * nc + col) * 4 : 0x40000000;
  auto store_at = [&](int sl, int nm, int nc, int r, float v) {
    const int skip = (16 * nm + r) * row_bytes, left = M2 * row_bytes - skip;
    const __amdgpu_buffer_rsrc_t ro =
        raw_buffer(reinterpret_cast<const char*>(a.out) + (int64_t)sl * M2 * row_bytes + skip, left > 0 ? left : 0);
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), ro, ofs[nc], 0, 0);
  };
  clear();
  v4f held[NC];                                                          // (tiles of 16 rows) y of an even tile
#pragma unroll
  for (int nc = 0; nc < NC; ++nc) held[nc] = (v4f){0.f, 0.f, 0.f, 0.f};
  bool pending = false;
  int pending_slab = 0;
  auto store_slab = [&]() {
#pragma unroll
    for (int nm = 0; nm < NM; ++nm)
#pragma unroll
      for (int nc = 0; nc < NC; ++nc)
#pragma unroll
        for (int r = 0; r < 4; ++r) store_at(pending_slab, nm, nc, r, value(nm, nc, r));
    clear();
  };
  // One tile, from the registers of set `set`; its tile of kAhead tiles later goes in flight under it.  Loads retire in
  // order, so what the next tile waits for (its support) is requested before those.
  auto tile = [&](auto set) {
    constexpr int D = decltype(set)::value;
    const uint32_t e_base = (uint32_t)slab * slab_elems + (uint32_t)(ts * R * K);   // I < 2^31
    const int rows = I2 - ts * R, n_e = (rows < R ? rows : R) * K;
    wave_sync();                                                         // previous tile's LDS reads are done
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
    if (pending) {                                                       // (stores here, not in front of the wait above)
      store_slab();
      pending = false;
    }
    const int32_t cur_om = my_om;
    uint32_t nj0 = 0, nj1 = 0;
    if constexpr (!ONE) {
      set_fetch(kAhead == 1 ? s1 : s2, kAhead == 1 ? t1 : t2);
      nj0 = __builtin_amdgcn_readfirstlane(nj0v);
      nj1 = s1 < a.nslabs ? __builtin_amdgcn_readfirstlane(nj1v) : nj0;
      issue_support(nj0, nj1);
      range_of(s2, t2, nj0v, nj1v);
    }
    wave_sync();
    {                                                                    // Sparse(G, Omega): hand the values over, then remove them
      auto take = [&](uint32_t j, int32_t oj) {
        const uint32_t e = (uint32_t)oj - e_base;
        float* p = sX + ES * (e + (pad ? div_magic(e, a.magicK) : 0u));
        a.gs[cj0 + j] = load_elem<DT>(p, 0);
        if (keep) return;
        if constexpr (DT == TGRAD_C64) *reinterpret_cast<float2*>(p) = make_float2(0.f, 0.f);
        else *reinterpret_cast<uint32_t*>(p) = 0u;
      };
      const uint32_t cnt = cj1 - cj0;
      if ((uint32_t)lane < cnt) take((uint32_t)lane, cur_om);
      if (cnt > 64u)
        for (uint32_t j = 64u + lane; j < cnt; j += 64) take(j, a.omega[cj0 + j]);
    }
    wave_sync();
    __builtin_amdgcn_s_setprio(1);
    // The next tile's loads go between the products of the first contraction: a load waits at issue until the memory
    // pipeline takes it, and there that wait lies under matrix instructions.
    constexpr int kTerms = DT == TGRAD_C64 ? 6 : 3, kSlots = QN * kTerms, kPer = (TB + kSlots - 1) / kSlots;
    constexpr int H = R / 16;
    v4f y[H][NC];
    auto issue_at = [&](int slot) {
#pragma unroll
      for (int i = 0; i < kPer; ++i)
        if (slot * kPer + i < TB) {
          __builtin_amdgcn_sched_barrier(0);
          issue_piece(raw[D], slot * kPer + i);
          __builtin_amdgcn_sched_barrier(0);
        }
    };
    // (The loads lie in the first half, which every tile has: a load on one of two paths would make the compiler wait for it
    // wherever they meet.)
#pragma unroll
    for (int h = 0; h < H; ++h) {
#pragma unroll
      for (int nc = 0; nc < NC; ++nc) y[h][nc] = (v4f){0.f, 0.f, 0.f, 0.f};
      if (h == 0 || rows > 16 * h) {                                     // (wave-uniform)
        v4f yl[NC];                                                      // the small terms have sums of their own
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) yl[nc] = (v4f){0.f, 0.f, 0.f, 0.f};
        const float* xa = sX + (16 * h + col) * stride + ES * grp;
#pragma unroll
        for (int q = 0; q < QN; ++q) {
          Split8 x;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float* p = xa + ES * (16 * q + 4 * j);
            if constexpr (DT == TGRAD_C64) split_at(x, j, *reinterpret_cast<const float2*>(p));
            else x.h[j] = *reinterpret_cast<const uint32_t*>(p);
          }
          const u32v4* cp = sC + q * (NC * 192) + lane;
          u32v4 c[NC];
          auto operand = [&](int k) {
#pragma unroll
            for (int nc = 0; nc < NC; ++nc) {
              if constexpr (kInLds) c[nc] = cp[nc * 192 + k * 64];
              else c[nc] = k == 0 ? cq[q][nc].h : k == 1 ? cq[q][nc].m : cq[q][nc].l;
            }
          };
          auto product = [&](int slot, const u32v4& xv, v4f* to) {
#pragma unroll
            for (int nc = 0; nc < NC; ++nc) to[nc] = mfma_bf(xv, c[nc], to[nc]);
            if (!ONE && h == 0) issue_at(kTerms * q + slot);
          };
          operand(2);
          product(0, x.h, yl);
          operand(1);
          if constexpr (DT == TGRAD_C64) {
            product(1, x.m, yl);
            product(2, x.h, yl);
            operand(0);
            product(3, x.l, yl);
            product(4, x.m, yl);
            product(5, x.h, y[h]);
          } else {
            product(1, x.h, yl);
            operand(0);
            product(2, x.h, y[h]);
          }
        }
        if constexpr (REST > 0) {
          const float2 xv = load_elem<DT>(xa + 16 * ES * QN, 0);
#pragma unroll
          for (int nc = 0; nc < NC; ++nc) {
            y[h][nc] = mfma16(xv.x, crest[nc].x, y[h][nc]);
            yl[nc] = mfma16(xv.y, crest[nc].y, yl[nc]);
          }
        }
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) y[h][nc] += yl[nc];
      }
    }
    auto second = [&](const v4f* lo, const v4f* hi) {
      Split8 b[NC];
#pragma unroll
      for (int nc = 0; nc < NC; ++nc)
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          split_at(b[nc], d, make_float2(lo[nc][2 * d], lo[nc][2 * d + 1]));
          split_at(b[nc], 2 + d, make_float2(hi[nc][2 * d], hi[nc][2 * d + 1]));
        }
      const u32v4* ft = sT + (size_t)(R == 32 ? ts : ts >> 1) * (NM * kHeadItem) + lane;
#pragma unroll
      for (int nm = 0; nm < NM; ++nm) {
        const u32v4* p = ft + nm * kHeadItem;
        mfma_split<NC>(da[nm], ONE ? own_r[ONE ? nm : 0] : Split8{p[0], p[64], p[128]}, b);
        mfma_split<NC>(db[nm], ONE ? own_i[ONE ? nm : 0] : Split8{p[192], p[256], p[320]}, b);
      }
    };
    if constexpr (R == 32) {
      second(y[0], y[1]);
    } else {
      // tiles of 16 rows: an even one of a slab that is walked waits for its neighbour
      const bool odd = ts & 1, paired = odd && !split;
      if (odd || split || ts == S - 1) {                                 // (wave-uniform)
        v4f lo[NC], hi[NC];
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) {
          const v4f none = (v4f){0.f, 0.f, 0.f, 0.f};
          lo[nc] = paired ? held[nc] : odd ? none : y[0][nc];
          hi[nc] = odd ? y[0][nc] : none;
        }
        second(lo, hi);
      } else {
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) held[nc] = y[0][nc];
      }
    }
    if constexpr (!ONE) issue_lone(lone[D]);
    __builtin_amdgcn_s_setprio(0);
    if (!split && ts == S - 1) {
      pending = true;
      pending_slab = slab;
    }
    slab = s1;
    ts = t1;
    s1 = s2;
    t1 = t2;
    if (s2 < a.nslabs) advance(s2, t2);
    cj0 = nj0;
    cj1 = nj1;
  };
  for (int base = (int)blockIdx.x;;) {
    while (slab < a.nslabs) {
      tile(std::integral_constant<int, 0>());
      if constexpr (ONE) break;
      if constexpr (kAhead > 1) {
        if (slab >= a.nslabs) break;                                       // (out of the loop: no path on which set 0 was just requested)
        tile(std::integral_constant<int, kAhead - 1>());
      }
    }
    if (pending) store_slab();
    if (split) {                                                           // the wavefronts' parts of the slab, in order
      __syncthreads();
      constexpr int kPart = NM * NC * 4 * 64;
#pragma unroll
      for (int nm = 0; nm < NM; ++nm)
#pragma unroll
        for (int nc = 0; nc < NC; ++nc)
#pragma unroll
          for (int r = 0; r < 4; ++r) sX[((nm * NC + nc) * 4 + r) * 64 + lane] = value(nm, nc, r);
      __syncthreads();
#pragma unroll
      for (int e = 0; e < NM * NC * 4; ++e)
        if (e % W == wave) {
          float v = 0.f;
          for (int w = 0; w < W; ++w) v += smem[w * slice + e * 64 + lane];
          store_at(base, e / (4 * NC), (e >> 2) % NC, e & 3, v);
        }
      static_assert(kPart <= 1024, "head_slice");
    }
    // With coefficients in LDS a workgroup stays for several shared slabs: its tables leave few of its kind to a compute unit
    // (head_mode).  Where they are light the code for it costs more than it saves (16x16x8x5 15.4 -> 15.9).
    if constexpr (MODE != HEAD_MANY || !head_many_coefs(T4, NC)) {
      break;
    } else {
      base += (int)gridDim.x;
      if (!split || base >= a.nslabs) break;
      slab = wave < S ? base : a.nslabs;
      ts = wave;
      s1 = slab;
      t1 = ts;
      if (slab < a.nslabs) advance(s1, t1);
      s2 = s1;
      t2 = t1;
      if (s1 < a.nslabs) advance(s2, t2);
      __syncthreads();                                                       // the sums are read
      // Commits leave the pads of the rows out: zeros again where the sums lay.  (A float32 read as a bf16 pair is an
      // infinity or NaN once in 256, which the zero coefficients it meets would not take out of the product.)
      if (pad) {
#pragma unroll
        for (int e = 0; e < NM * NC * 4; ++e) sX[e * 64 + lane] = 0.f;
      }
      issue_tile(raw[0], lone[0], slab, ts);
      range_of(slab, ts, cj0v, cj1v);
      range_of(s1, t1, nj0v, nj1v);
      first_support();
      if constexpr (kAhead > 1) issue_tile(raw[kAhead - 1], lone[kAhead - 1], s1, t1);
      clear();
    }
  }
}

// ---- k_tail -------------------------------------------------------------------------------------
// Stage A  D'[(m3, p), i2] = sum_m2 Y1[m2, (m3, p)] U2[i2, m2]:  A operand = rows of the slab's Y1 (registers, parts
//   chosen per p once per slab), B operand = U2 from the LDS table; lane (i2 = c, g) then holds (re, im) of elements
//   m3 = 8 nc + 2 g + {0, 1} of row i2 - the A operand of stage B as it stands.
// Stage B  tile[i2, column] = sum_m3 D'[.., i2] (c_alpha U3)[column, m3], 16 columns at a time, coefficients in
//   registers; the flat image of the tile in LDS then takes the sparse entries and is streamed into W.
// A last mode of 8 m + 1 complex columns has its last column done by vector arithmetic, not by a tile of its own.
// Both on split bf16 operands (device_common.h).  Stage A: slot 2 j + u of lane (c, g) is part u of m2 = 16 q + 4 j + g;
// stage B: slot 4 nc + r is register r of D' tile nc.
constexpr int tail_rows(int CT) { return CT <= 4 ? 32 : 16; }
// Coefficients of more than four operands' worth of columns leave no registers for a next tile: they are then kept in LDS,
// which the kernel has to spare (a tile reads CT x 3 KB of them per 16 rows), unless there is no next tile (ONE).
constexpr bool tail_coef_lds(int CT, int NC) { return CT * NC > 4; }
constexpr int tail_pieces(int CT) { return CT == 2 ? 5 : CT == 3 ? 7 : 9; }   // complex64 pieces per lane of a tile
__host__ __device__ constexpr int tail_slice(int M, int R) { return (R * 2 * M + 3) & ~3; }

// Tiles in flight per wavefront: two where the registers hold them (see head_ahead; 6400 slabs of 100x36, r 16,8 75 / 73 us,
// the others of those the same)
constexpr int tail_ahead(int CT, int NC, int SA) { return SA == 8 && NC == 2 ? 1 : CT == 9 || NC == 2 ? 2 : 1; }

// Whether a kernel has the code for slabs that several wavefronts walk together (launch_tail has the rule).
constexpr bool tail_shares(int WDT, int CT) { return WDT == TGRAD_C64 && CT > 2; }

struct TailArgs {
  const float2* y1;             // (nslabs, K2, K) complex
  const float2* U2;             // (I2, K2)
  const float2* U3;             // (M, K)
  void* w;
  int K, M, I2, K2, S, nslabs;
  int split;                    // 1: single tiles are dealt to the wavefronts; 0: whole slabs; 2, 4: slabs that many wavefronts walk
                                // together, tile by tile in turn (divides W and S)
  float decay, c_alpha;
};

// ONE: a workgroup is one wavefront with one tile
// (of a class with many coefficients, tail_coef_lds): no table, no next tile
template <int WDT, int CT, int NC, int SA, bool ONE>
__global__ __launch_bounds__(64 * kMaxWaves, 2) void k_tail(TailArgs a, SparseAdam sp) {
  typedef WStore<WDT> WS;
  typedef typename WS::raw wraw;
  constexpr int R = tail_rows(CT);
  constexpr int kPre = WS::kElems == 2 ? tail_pieces(CT) : (tail_pieces(CT) + 1) / 2;
  constexpr int kElem = 16 / WS::kElems;                                 // bytes of an element of W
  extern __shared__ float smem[];
  const int K = a.K, M = a.M, I2 = a.I2, K2 = a.K2, S = a.S;
  const int N2 = 2 * M;
  const int slice = tail_slice(M, R);
  const int W = (int)blockDim.x >> 6;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4, part = lane & 1;
  float* sD = smem + wave * slice;
  u32v4* sT = reinterpret_cast<u32v4*>(smem + W * slice);                // U2 in operand order [16 rows][quad][h, m, l][lane]
  constexpr int KA = SA > 4 ? 2 : 1;                                     // quads of K2
  const bool vtail = (N2 & 15) == 2;
  const int NT = vtail ? N2 >> 4 : (N2 + 15) >> 4;                       // column tiles (<= CT: host)
  constexpr bool kShare = tail_shares(WDT, CT);
  const bool split = kShare ? a.split == 1 : a.split != 0;
  const int nw = (int)gridDim.x * W;
  int block = (int)blockIdx.x;
  if (kShare && a.split > 1 && W == 4 && (int)gridDim.x % (8 * a.split) == 0) {
    // slabs on the XCD on which k_head has them, four to a workgroup: its L2 has the support's places and values (launch_tail)
    const int in = block % (8 * a.split);
    block += a.split * (in & 7) + (in >> 3) - in;
  }
  const int first = block * W + wave;
  const int share = kShare ? a.split >> 1 : 0, every = kShare && share ? a.split : 1, ts0 = kShare ? wave & (every - 1) : 0;
  int slab = split ? first / S : first >> share, ts = split ? first - slab * S : ts0;
  auto advance = [&](int& sl, int& t) {
    if (split) {
      t += nw;
      sl += t / S;
      t = t % S;
    } else if (t + every < S) {
      t += every;
    } else {
      t = ts0;
      sl += nw >> share;
    }
  };
  const uint32_t slab_elems = (uint32_t)(I2 * M);
  constexpr int kAhead = ONE ? 1 : tail_ahead(CT, NC, SA);
  wraw wpre[kAhead][kPre];                                               // the tiles in flight
  uint32_t wl0[kAhead], wl1[kAhead];                                     // elements past the last whole piece of a tile
  auto tile_elems = [&](int t) -> int { return (I2 - t * R < R ? I2 - t * R : R) * M; };
  auto tile_addr = [&](int sl, int t) -> char* {
    return reinterpret_cast<char*>(a.w) + ((uint64_t)(uint32_t)sl * slab_elems + (uint32_t)(t * R * M)) * (uint64_t)kElem;
  };
  auto issue_w = [&](wraw* to, uint32_t& l0, uint32_t& l1, int sl, int t) {                                    // (no tile: empty descriptors)
    const bool ok = sl < a.nslabs;
    const int n = ok ? tile_elems(t) : 0, n4 = n / WS::kElems;
    const char* base = ok ? tile_addr(sl, t) : reinterpret_cast<const char*>(a.w);
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
  u32x2 my_g, my_m;
  uint32_t my_v = 0;
  auto issue_sparse = [&](uint32_t j0, uint32_t j1) {                    // the first 64 entries of a tile
    const uint32_t n = j1 - j0 < 64u ? j1 - j0 : 64u;
    my_om = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(raw_buffer(sp.omega + j0, n * 4u), lane * 4, 0, 0);
    my_g = __builtin_amdgcn_raw_buffer_load_b64(raw_buffer(sp.gs + j0, n * 8u), lane * 8, 0, 0);
    my_m = __builtin_amdgcn_raw_buffer_load_b64(raw_buffer(sp.ms + j0, n * 8u), lane * 8, 0, 0);
    my_v = __builtin_amdgcn_raw_buffer_load_b32(raw_buffer(sp.vs + j0, n * 4u), lane * 4, 0, 0);
  };
  float2 y[SA][NC];
  auto fetch_y = [&](int sl) {                                           // rows / columns past the end meet zero coefficients
    const float2* yp = a.y1 + (int64_t)sl * K2 * K;
#pragma unroll
    for (int s = 0; s < SA; ++s)
#pragma unroll
      for (int nc = 0; nc < NC; ++nc) {
        const int m2 = 4 * s + grp, m3 = 8 * nc + (col >> 1);
        y[s][nc] = yp[(m2 < K2 ? m2 : K2 - 1) * K + (m3 < K ? m3 : K - 1)];
      }
  };
  const uint32_t vzero = (uint32_t)opaque_zero();
  auto range_of = [&](int sl, int t, uint32_t& j0, uint32_t& j1) {
    const uint32_t* tsb = sp.tile_start + (sl < a.nslabs ? (int64_t)sl * S + t : 0);
    j0 = tsb[vzero];
    j1 = tsb[vzero + 1];
  };
  // ---- prologue: the first tile of W, its operands and the tables go in flight ----
  int nslab = slab, nts = ts;                                            // the tile after this one, the one after that
  if (slab < a.nslabs) advance(nslab, nts);
  int s2 = nslab, t2 = nts;
  if (nslab < a.nslabs) advance(s2, t2);
#pragma unroll
  for (int d = 0; d < kAhead; ++d) wl0[d] = wl1[d] = 0;
  issue_w(wpre[0], wl0[0], wl1[0], slab, ts);
  uint32_t cj0v, cj1v, nj0v, nj1v;
  range_of(slab, ts, cj0v, cj1v);
  if constexpr (!ONE) range_of(nslab, nts, nj0v, nj1v);
  fetch_y(slab < a.nslabs ? slab : 0);
  const FactorRef fU3 = factor_ref(a.U3, (int64_t)M * K), fU2 = factor_ref(a.U2, (int64_t)I2 * K2);
  // (c_alpha U3)[column][8 nc + 2 g + u], dword 2 nc + u
  constexpr bool kInLds = !ONE && tail_coef_lds(CT, NC);
  Split8 cf[kInLds ? 1 : CT];
  u32v4* sC = sT + ((I2 + 15) >> 4) * (KA * 192);
  float2 ct[NC][2];
#pragma unroll
  for (int nc = 0; nc < NC; ++nc)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int k = 8 * nc + 2 * grp + u;
#pragma unroll
      for (int i = 0; i < CT; ++i) {
        const int m = (16 * i + col) >> 1;
        if constexpr (!kInLds) {
          const float2 f = factor_entry(fU3, m, k, K, k < K && m < M);
          split_at(cf[i], 2 * nc + u, column_coef(make_float2(a.c_alpha * f.x, a.c_alpha * f.y), part));
        }
      }
      const float2 f = factor_entry(fU3, M - 1, k, K, k < K);
      ct[nc][u] = make_float2(a.c_alpha * f.x, a.c_alpha * f.y);
    }
  auto table_load = [&](int e, float2* u) {
    const int l = e & 63, q = (e >> 6) % KA, i2 = 16 * ((e >> 6) / KA) + (l & 15);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m2 = 16 * q + 4 * j + (l >> 4);
      u[j] = factor_entry(fU2, i2, m2, K2, i2 < I2 && m2 < K2);
    }
  };
  Split8 own[ONE ? R / 16 : 1][ONE ? KA : 1];                            // (ONE) the table's rows of the tile
  if constexpr (ONE) {
    float2 u[R / 16][KA][4];
#pragma unroll
    for (int h = 0; h < R / 16; ++h)
#pragma unroll
      for (int q = 0; q < KA; ++q) table_load(((ts * (R / 16) + h) * KA + q) * 64 + lane, u[h][q]);
#pragma unroll
    for (int h = 0; h < R / 16; ++h)
#pragma unroll
      for (int q = 0; q < KA; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) split_at(own[h][q], j, u[h][q][j]);
  } else {
    for (int e = tid; e < ((I2 + 15) >> 4) * KA * 64; e += (int)blockDim.x) {
      float2 u[4];
      table_load(e, u);
      Split8 f;
#pragma unroll
      for (int j = 0; j < 4; ++j) split_at(f, j, u[j]);
      u32v4* p = sT + (e >> 6) * 192 + (e & 63);
      p[0] = f.h;
      p[64] = f.m;
      p[128] = f.l;
    }
  }
  if constexpr (kInLds) {
    constexpr int kItems = 3;                                            // (as in k_head)
    for (int i0 = wave; i0 < CT; i0 += kItems * W) {
      float2 f[kItems][2 * NC];
#pragma unroll
      for (int u = 0; u < kItems; ++u) {
        const int m = (16 * (i0 + u * W) + col) >> 1;
#pragma unroll
        for (int d = 0; d < 2 * NC; ++d) {
          const int k = 8 * (d >> 1) + 2 * grp + (d & 1);
          f[u][d] = factor_entry(fU3, m, k, K, k < K && m < M);
        }
      }
#pragma unroll
      for (int u = 0; u < kItems; ++u)
        if (i0 + u * W < CT) {
          Split8 c = {};
#pragma unroll
          for (int d = 0; d < 2 * NC; ++d)
            split_at(c, d, column_coef(make_float2(a.c_alpha * f[u][d].x, a.c_alpha * f[u][d].y), part));
          u32v4* p = sC + (i0 + u * W) * 192 + lane;
          p[0] = c.h;
          p[64] = c.m;
          p[128] = c.l;
        }
    }
  }
  uint32_t cj0 = __builtin_amdgcn_readfirstlane(cj0v), cj1 = __builtin_amdgcn_readfirstlane(cj1v);
  if (slab >= a.nslabs) cj1 = cj0;
  issue_sparse(cj0, cj1);
  if constexpr (kAhead > 1) issue_w(wpre[kAhead - 1], wl0[kAhead - 1], wl1[kAhead - 1], nslab, nts);
  if constexpr (!ONE) __syncthreads();                                   // the only workgroup barrier
  bool fresh = true;                                                     // y as loaded, not yet in operand form
  Split8 ya[KA][NC];
  auto tile = [&](auto set) {
    constexpr int D = decltype(set)::value;
    const uint32_t w_base = (uint32_t)slab * slab_elems + (uint32_t)(ts * R * M);
    const int n_w = tile_elems(ts), n4 = n_w / WS::kElems, rows = I2 - ts * R;
    char* w_tile = tile_addr(slab, ts);
    if (fresh) {
      // row (m3, p): re(u y) = ur yr - ui yi, im(u y) = ur yi + ui yr
#pragma unroll
      for (int s = 0; s < 4 * KA; ++s)
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) {
          const float2 v = s < SA ? y[s < SA ? s : 0][nc] : make_float2(0.f, 0.f);
          split_at(ya[s >> 2][nc], s & 3, part ? make_float2(v.y, v.x) : make_float2(v.x, -v.y));
        }
      fresh = false;
    }
    wave_sync();                                                         // previous tile's LDS reads are done
#pragma unroll
    for (int h = 0; h < R / 16; ++h) {
      if (h == 0 || rows > 16 * h) {                                     // (wave-uniform)
        v4f dz[NC];
#pragma unroll
        for (int nc = 0; nc < NC; ++nc) dz[nc] = (v4f){0.f, 0.f, 0.f, 0.f};
        const u32v4* ft = sT + (size_t)(ts * (R / 16) + h) * (KA * 192) + lane;
#pragma unroll
        for (int q = 0; q < KA; ++q)
          mfma_split_b<NC>(dz, ya[q], ONE ? own[ONE ? h : 0][ONE ? q : 0] : Split8{ft[q * 192], ft[q * 192 + 64], ft[q * 192 + 128]});
        Split8 za;
#pragma unroll
        for (int nc = 0; nc < NC; ++nc)
#pragma unroll
          for (int u = 0; u < 2; ++u) split_at(za, 2 * nc + u, make_float2(dz[nc][2 * u], dz[nc][2 * u + 1]));
        float* sR = sD + (16 * h + 4 * grp) * N2 + col;
#pragma unroll
        for (int i = 0; i < CT; ++i) {
          if (i < NT) {                                                  // (wave-uniform)
            v4f o = (v4f){0.f, 0.f, 0.f, 0.f};
            const Split8 b = kInLds ? Split8{sC[i * 192 + lane], sC[i * 192 + lane + 64], sC[i * 192 + lane + 128]}
                                    : cf[kInLds ? 0 : i];
            if constexpr (NC == 1) mfma_split_half(o, za, b);
            else mfma_split<1>(&o, za, &b);
            if (16 * i + col < N2) {
#pragma unroll
              for (int r = 0; r < 4; ++r) sR[r * N2 + 16 * i] = o[r];   // (rows past the slab's end: written, not streamed)
            }
          }
        }
        if (vtail) {
          float pre = 0.f, pim = 0.f;
#pragma unroll
          for (int nc = 0; nc < NC; ++nc)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const float zr = dz[nc][2 * u], zi = dz[nc][2 * u + 1];
              pre += zr * ct[nc][u].x - zi * ct[nc][u].y;
              pim += zr * ct[nc][u].y + zi * ct[nc][u].x;
            }
          pre += __shfl_xor(pre, 16, 64);
          pim += __shfl_xor(pim, 16, 64);
          pre += __shfl_xor(pre, 32, 64);
          pim += __shfl_xor(pim, 32, 64);
          if (grp == 0)
            *reinterpret_cast<float2*>(&sD[(16 * h + col) * N2 + N2 - 2]) = make_float2(pre, pim);
        }
      }
    }
    if (!ONE && nslab < a.nslabs && nslab != slab) {                             // (wave-uniform) the next tile opens another slab
      fetch_y(nslab);
      fresh = true;
    }
    wave_sync();
    // ---- AdamUpdate on the sparse values that live in this tile; add lambda N_S into the tile ----
    {
      const uint32_t cnt = cj1 - cj0;
      if ((uint32_t)lane < cnt)
        sparse_adam_entry(sp, cj0 + lane, my_om, make_float2(__uint_as_float(my_g.x), __uint_as_float(my_g.y)),
                          make_float2(__uint_as_float(my_m.x), __uint_as_float(my_m.y)), __uint_as_float(my_v),
                          (int64_t)w_base, sD);
      if (cnt > 64u)                                                     // rare: more than 64 entries in one tile
        for (uint32_t j = cj0 + 64u + lane; j < cj1; j += 64)
          sparse_adam_entry(sp, j, sp.omega[j], sp.gs[j], sp.ms[j], sp.vs[j], (int64_t)w_base, sD);
    }
    wave_sync();
    // ---- stream the tile into W ----
#pragma unroll
    for (int i = 0; i < kPre; ++i) claim_raw(wpre[D][i]);
#pragma unroll
    for (int k = 0; k < (kPre + 3) / 4; ++k) {
      const int left = n4 * 16 - k * 4096;
      const __amdgpu_buffer_rsrc_t r = raw_buffer(w_tile + k * 4096, (uint32_t)(left > 0 ? left : 0));
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
          *reinterpret_cast<float2*>(w_tile + (int64_t)e * kElem) =
              make_float2(a.decay * __uint_as_float(wl0[D]) + sD[2 * e], a.decay * __uint_as_float(wl1[D]) + sD[2 * e + 1]);
        else
          *reinterpret_cast<uint32_t*>(w_tile + (int64_t)e * kElem) =
              WStore<TGRAD_CBF16>::one(wl0[D], sD[2 * e], sD[2 * e + 1], a.decay);
      }
    }
    if constexpr (ONE) return;
    // ---- the next tiles go in flight: the support first, which the next tile waits for (loads retire in order) ----
    cj0 = __builtin_amdgcn_readfirstlane(nj0v);
    cj1 = nslab < a.nslabs ? __builtin_amdgcn_readfirstlane(nj1v) : cj0;
    issue_sparse(cj0, cj1);
    range_of(s2, t2, nj0v, nj1v);
    issue_w(wpre[D], wl0[D], wl1[D], kAhead == 1 ? nslab : s2, kAhead == 1 ? nts : t2);
    slab = nslab;
    ts = nts;
    nslab = s2;
    nts = t2;
    if (s2 < a.nslabs) advance(s2, t2);
  };
  while (slab < a.nslabs) {
    tile(std::integral_constant<int, 0>());
    if constexpr (ONE) break;
    if constexpr (kAhead > 1) {
      if (slab >= a.nslabs) break;                                       // (out of the loop: no path on which set 0 was just requested)
      tile(std::integral_constant<int, kAhead - 1>());
    }
  }
}

// ---- host side ----------------------------------------------------------------------------------

int steps_class(int K) {                        // k_head's T4
  const int t = (K + 3) / 4;
  if (K <= 33) return t <= 3 ? 3 : t <= 5 ? 5 : t <= 7 ? 7 : 9;
  return t <= 13 ? 13 : 17;
}
int columns_class(int M) { return M <= 17 ? 2 : M <= 25 ? 3 : M <= 33 ? 4 : 9; }   // k_tail's CT
int step_class(int K2) { return K2 <= 8 ? 2 : K2 <= 16 ? 4 : 8; }                  // k_tail's SA

size_t head_lds(int mode, int W, int ES, int K, int M, int I2, int M2) {
  const int t4 = steps_class(K), nc = M <= 8 ? 1 : 2;
  const size_t slices = (size_t)W * head_slice(ES, K, t4) * 4;
  if (mode == HEAD_ONE) return slices;
  return (mode == HEAD_MANY && head_coef_lds(t4, nc) ? (size_t)head_quads(t4) * nc * 3072 : 0) + slices + (size_t)((I2 + 31) / 32) * ((M2 + 15) / 16) * kHeadItem * 16;
}
size_t tail_lds(int W, int M, int I2, int K2, int K, bool one = false) {
  const int ct = columns_class(M);
  if (one) return (size_t)tail_slice(M, end_tile_rows(M)) * 4;
  return (size_t)W * tail_slice(M, end_tile_rows(M)) * 4 + (size_t)((I2 + 15) / 16) * (K2 > 16 ? 2 : 1) * 3072 +
         (tail_coef_lds(ct, K <= 8 ? 1 : 2) ? (size_t)ct * 3072 : 0);
}

// From this many slabs on a wavefront takes whole ones (one wavefront per SIMD of the chip).
constexpr int64_t kWholeSlabs = 1024;

// Workgroups of a launch over `units` wavefronts' worth of work
template <typename Kern>
unsigned end_grid(Kern kern, int W, size_t lds, int64_t units) {
  const int64_t groups = (units + W - 1) / W, cap = (int64_t)compute_units() * resident_blocks(kern, 64 * W, lds, 8);
  return (unsigned)(groups < cap ? groups : cap);
}

}  // namespace

int end_tile_rows(int K) { return K <= 33 ? 32 : 16; }

// Which shapes take the two kernels: K = extent of the last mode, r its rank, I2 / r2 extent and rank of mode N-1.
// Slabs of fewer than four rows would leave seven eighths of every tile empty (and need a support offset for every few
// entries): they stay with the kernels that cut the tensor into tiles of 32 rows wherever a slab ends.
bool ends_kernel_fits(int K, int r, int I2, int r2) {
  if (K < 2 || K > 68 || r > 16 || r2 > 32 || I2 < 4 || I2 > TGRAD_MAX_EXTENT) return false;
  return head_lds(HEAD_MANY, 4, 2, K, r, I2, r2) <= kLdsLimit && tail_lds(4, K, I2, r2, r) <= kLdsLimit;
}

// Where the 32 x 32 kernels, if the shape suits them (512 slabs of whole 32-row tiles), are the better ones: both ranks in the
// upper half of a 32-wide tile, or a table of conj(U2) that leaves one workgroup per compute unit, and not yet the slabs for
// these kernels to fill the chip with.  Whole step, us, those / these: r 32,16 or 17,9 behind 8,8
//   512 slabs: 32x17 21.1 / 21.6, 32x33 26.0 / 29.3, 128x65 60.5 / 57.3;  1024: 32x33 30.0 / 31.1, 128x65 71.6 / 82.5;
//   2048: 32x17 32.5 / 31.2, 32x33 48.7 / 43.5, 128x65 117 / 115;  4096: 49 / 42, 66 / 60, 200 / 200;
//   16384: 123 / 90, 158 / 139, 706 / 699;      256x13, r 20,5: 1024 slabs 60 / 52, 4096 166 / 97.
bool wide_tiles_pay(int r, int I2, int r2, int64_t nslabs) {
  if (r > 8 && r2 > 16) return nslabs < 2048;
  return nslabs < 1024 && ((I2 + 31) / 32) * ((r2 + 15) / 16) * kHeadItem * 16 > (int)kLdsLimit / 2;
}

// ... and which of those it pays for.  A tile costs a wavefront the same few round trips and whole 16-row halves of matrix
// work however few rows it holds, and past 8192 slabs (two or more for every resident wavefront) the tiles of short slabs
// follow each other; the separate kernels per mode take flat tiles of 32 rows wherever a slab ends, for one more launch
// each way and one more trip of the mode-N result (r numbers per row) through memory.  (Slabs of whole 32-row tiles, which
// the 32 x 32 kernels take as well, are not asked about: these are faster there whatever the rank.)  With S tiles of H halves in a slab
// of I2 rows, both sides in the same units (fitted to 2400 measured pairs of whole steps; the worst choice loses 17 %).
// Whole step, us, these kernels / the separate ones, slabs of I2 x K with ranks a quarter of that:
//   16384 slabs: 4x5 41 / 32, 8x5 41 / 36, 16x5 42 / 42, 4x17 45 / 36, 8x17 47 / 46, 12x17 50 / 56, 4x65 89 / 71, 8x65 95 / 101;
//   65536: 4x5 84 / 45, 8x5 88 / 60, 16x5 93 / 91, 24x5 114 / 118, 36x5 181 / 162, 8x9 93 / 74, 16x9 103 / 107, 8x17 108 / 96,
//   12x17 118 / 123, 6x33 144 / 127, 8x33 153 / 151, 5x50 233 / 174;  262144: 4x3 252 / 96, 8x9 286 / 192, 28x2 341 / 367;
//   4096 slabs: 4x5 24 / 27, 8x33 32 / 33, 36x5 31 / 33 (the saved launches win).
// r: 65536 slabs of 12x9 with r = 1 95 / 82, r = 6 109 / 115, r = 9 126 / 143.
bool ends_kernel_pays(int K, int r, int I2, int r2, int64_t nslabs) {
  // (Few slabs of the longest, with two tiles of their rank: eight tiles of 32 rows with a workgroup for each slab or a table
  // for few of them, or thirteen and more of 16 with two column tiles, are not worth it.  27 slabs of 232x15, r 32,2 26 / 24,
  // 76 of 246x30, r 21,8 34 / 32, 120 of 232x13, r 24,9 49 / 44, 96 of 204x56, r 27,16 48 / 44; but 84 of 188x20, r 30,7 26 / 30, 68 of 206x67, r 32,11 47 / 47, 39 of 146x62,
  // r 18,7 25 / 37, 126 of 242x26, r 25,15 34 / 40.)
  if (nslabs < 128 && r2 > 16 && (K <= 33 ? I2 > 224 && K > 12 && (r <= 8 || K <= 20) : I2 > 192 && K > 52 && r > 8)) return false;
  // (... nor with four wavefronts for all of a compute unit while a fourth round is begun and not filled: 816 slabs of 247x60,
  // r 26,12 135 / 130, 900 of 220x50 122 / 119, 909 of 236x51, r 30,12 127 / 122; but 625 of 250x65, r 32,16 115 / 121, 1600
  // of 220x50 156 / 165.)
  if (nslabs >= 768 && nslabs < kWholeSlabs && r > 8 && head_lds(HEAD_MANY, 8, 2, K, r, I2, r2) > kLdsLimit) return false;
  if (nslabs < 8192) return true;
  const int R = end_tile_rows(K), S = (I2 + R - 1) / R, H = (I2 + 15) / 16;
  const int row = 25 + (K < 17 ? K : 17) + 5 * r;
  const int tiles = (nslabs < 16384 ? 35 : 50) * (6 * S + (r2 > 16 ? 9 : 5) * H);
  return I2 * (row < 70 ? row : 70) >= tiles;
}

namespace {

// (One class more: where slabs of four tiles meet two tiles of rank, its table leaves a compute unit one workgroup of four
// wavefronts.  390 slabs of 118x30, r 23,5 13.5 us, now 9.0; 780 of 100x29, r 32,8 25.6, now 14.3.)
constexpr bool head_has_one(int DT, int T4, int NC, int NM) {
  return head_many_coefs(T4, NC) || (DT == TGRAD_C64 && T4 >= 5 && NC == 1 && NM == 2);
}

// Which of the three HEAD_ modes, while slabs are too few for a wavefront to walk whole ones (us, k_head alone, r: ranks of
// the two modes; the last figure is the kernel on float32 instructions that these took the place of):
//   HEAD_ONE for slabs of up to four tiles, and of up to eight if all of them are resident at once (a workgroup of 5 to 8
//     wavefronts has two on some SIMD, so it is asked about as one of 8).  ONE / FEW / MANY / float32: 11x9x29, r 2,9
//     5.3 / 5.9 / 7.1 / 5.9; 42x42x44, r 13,14 6.6 / 7.4 / 8.7 / 7.3; 900 slabs of 42x44, r 32,12 16 / 22 / 20 / 18; 400 of 78x30,
//     r 27,12 11.9 / 12.6 / 14.0 / 13.8; but 306 slabs of six tiles, 82x49, r 6,9 15.5 / 13.0 / 13.5 / 12.6;
//   HEAD_FEW for complex64 G where two workgroups fit a compute unit, and for rows of up to 52 elements no more than three
//     slabs per compute unit.  FEW / MANY / float32: 380 slabs of 86x61, r 19,5 12.6 / 15.7 / 12.4; 484 of 79x39, r 19,9
//     14.4 / 17.8 / 13.9; 841 of 90x67, r 4,12 26.3 / 29.6 / 26.7; 688 of 99x50, r 32,16 25.2 / 28.7 / 27.0; but 936 of 100x43,
//     r 15,14 23.7 / 22.4 / 22.7; with one workgroup, 552 of 99x55, r 19,12 36 / 28 / 27; with bf16 G, which takes half the LDS
//     and three products of six, 784 of 77x63, r 22,11 24.3 / 22.4 / 29.1;
//   HEAD_MANY for the rest.
template <int DT, int T4, int NC, int NM>
int head_mode(int64_t nslabs, int S, int es, int K, int M, int I2, int M2) {
  if (!head_has_one(DT, T4, NC, NM) || nslabs >= kWholeSlabs) return HEAD_MANY;
  if (!head_many_coefs(T4, NC) && head_lds(HEAD_MANY, 4, es, K, M, I2, M2) <= kLdsLimit / 2) return HEAD_MANY;
  if (S <= 4) return HEAD_ONE;
  if constexpr (head_has_one(DT, T4, NC, NM)) {
    const auto one = k_head<DT, T4, NC, NM, HEAD_ONE>;
    const size_t lds = head_lds(HEAD_ONE, S, es, K, M, I2, M2);
    if (S <= kMaxWaves && allow_lds(one, lds) &&
        nslabs <= (int64_t)compute_units() * resident_blocks(one, 64 * kMaxWaves, lds))
      return HEAD_ONE;
  }
  const bool few = DT == TGRAD_C64 && head_coef_lds(T4, NC) && (T4 == 17 || nslabs <= 3 * (int64_t)compute_units());
  return few && head_lds(HEAD_FEW, 4, es, K, M, I2, M2) <= kLdsLimit / 2 ? HEAD_FEW : HEAD_MANY;
}

template <int DT, int T4, int NC, int NM, int MODE>
void launch_head_as(hipStream_t s, const HeadArgs& a, int W, size_t lds, int64_t nslabs) {
  const auto kern = k_head<DT, T4, NC, NM, MODE>;
  allow_lds(kern, lds);
  const bool stay = MODE == HEAD_MANY && (!a.split || head_many_coefs(T4, NC));
  const unsigned grid = stay ? end_grid(kern, W, lds, a.split ? nslabs * W : nslabs) : (unsigned)nslabs;
  kern<<<dim3(grid), dim3(64 * W), lds, s>>>(a);
}

template <int DT, int T4, int NC, int NM>
void launch_head_of(hipStream_t s, const HeadArgs& a, int64_t nslabs) {
  constexpr int es = DT == TGRAD_C64 ? 2 : 1;
  const int mode = head_mode<DT, T4, NC, NM>(nslabs, a.S, es, a.K, a.M, a.I2, a.M2);
  auto lds = [&](int W) { return head_lds(mode, W, es, a.K, a.M, a.I2, a.M2); };
  const int full = mode == HEAD_FEW || lds(4) <= kLdsLimit / 2 ? 4 : lds(8) <= kLdsLimit ? 8 : 4;
  const int W = mode == HEAD_ONE ? a.S : a.split ? (a.S < full ? a.S : full) : nslabs >= kWholeSlabs ? full : 1;
  if constexpr (head_has_one(DT, T4, NC, NM)) {
    if (mode == HEAD_ONE) return launch_head_as<DT, T4, NC, NM, HEAD_ONE>(s, a, W, lds(W), nslabs);
    if constexpr (DT == TGRAD_C64 && head_coef_lds(T4, NC))
      if (mode == HEAD_FEW) return launch_head_as<DT, T4, NC, NM, HEAD_FEW>(s, a, W, lds(W), nslabs);
  }
  launch_head_as<DT, T4, NC, NM, HEAD_MANY>(s, a, W, lds(W), nslabs);
}

}  // namespace

void launch_head(hipStream_t s, const void* g, int dtype, const int32_t* omega, const uint32_t* tile_start, float2* gs,
                 const float2* U3, int K, int M, const float2* U2, int I2, int M2, int64_t nslabs, bool keep, float2* out) {
  const int R = end_tile_rows(K), S = (I2 + R - 1) / R;
  const bool split = nslabs < kWholeSlabs && S > 1;
  HeadArgs a{g, omega, tile_start, gs, U3, U2, K, M, I2, M2, S, (int)nslabs, split ? 1 : 0, keep ? 1 : 0, magic_for(K),
             reinterpret_cast<float*>(out)};
  const int t4 = steps_class(K), nc = M <= 8 ? 1 : 2, nm = M2 <= 16 ? 1 : 2;
#define TGRAD_HEAD(DT_, T_, C_, M_) launch_head_of<DT_, T_, C_, M_>(s, a, nslabs)
#define TGRAD_HEAD_M(DT_, T_)                                                                                \
  do {                                                                                                       \
    if (nc == 1) { if (nm == 1) TGRAD_HEAD(DT_, T_, 1, 1); else TGRAD_HEAD(DT_, T_, 1, 2); }                 \
    else { if (nm == 1) TGRAD_HEAD(DT_, T_, 2, 1); else TGRAD_HEAD(DT_, T_, 2, 2); }                         \
  } while (0)
#define TGRAD_HEAD_T(DT_)                                                                                    \
  do {                                                                                                       \
    if (t4 == 3) TGRAD_HEAD_M(DT_, 3); else if (t4 == 5) TGRAD_HEAD_M(DT_, 5); else if (t4 == 7) TGRAD_HEAD_M(DT_, 7); \
    else if (t4 == 9) TGRAD_HEAD_M(DT_, 9); else if (t4 == 13) TGRAD_HEAD_M(DT_, 13); else TGRAD_HEAD_M(DT_, 17); \
  } while (0)
  if (dtype == TGRAD_C64) TGRAD_HEAD_T(TGRAD_C64); else TGRAD_HEAD_T(TGRAD_CBF16);
#undef TGRAD_HEAD_T
#undef TGRAD_HEAD_M
#undef TGRAD_HEAD
}

void launch_tail(hipStream_t s, const float2* y1, const float2* U3, int K, int M, const float2* U2, int I2, int K2,
                 int64_t nslabs, void* w, int wdtype, float decay, float c_alpha, const int32_t* omega,
                 const uint32_t* tile_start, const float2* gs, float2* ms, float* vs, float beta1, float beta2,
                 double inv_c1, double inv_c2, float eps, float c_lambda) {
  const int R = end_tile_rows(M), S = (I2 + R - 1) / R;
  // Single tiles are dealt to the wavefronts, and a slab's part of z fetched for every one of them, while slabs are few; of
  // five tiles and more also where whole ones leave most of the last round idle (2511 slabs for 2048 wavefronts), and for
  // complex64 W, up to 8 columns of rank and more than 17 of W, where such a fetch is little beside the tile.  Whole / dealt
  // (float32 operands, whole), us: 2511 slabs of 113x38, r 31,8 56 / 43 (48); 2304 of 110x35, r 5,15 44 / 34 (46); 2401 of
  // 84x53, r 25,11, bf16 W 41 / 37 (47); 6400 of 256x20, r 13,4 112 / 98 (112); 8991 of 192x28, r 17,6 163 / 153 (157); but
  // 3660 of 163x51, r 23,15, bf16 W 78 / 91; 8100 of 90x50, r 20,12 121 / 127; 6561 of 150x14, r 25,3 55 / 58; 12800 of
  // 250x12, r 20,4 142 / 156.
  const bool split = nslabs < kWholeSlabs ||
                     (S >= 5 && nslabs < (wdtype == TGRAD_C64 && K <= 8 && M > 17 ? 9 * kWholeSlabs : 5 * kWholeSlabs / 2));
  // Slabs are walked by two or four wavefronts of a workgroup together, in turn, where a slab has as many tiles (or a multiple): what
  // a workgroup has in flight then lies side by side, which is what the memory rewards (a stand-alone loop that updates 8 KB tiles
  // in place: 5.6 TB/s with wavefronts on slabs of their own, 5.2 with 16 KB tiles, 5.8 with wavefronts on consecutive
  // tiles).  Each of them fetches the slab's part of z, so for ranks of 17 and more in mode N-1 only slabs of many
  // tiles are shared; bf16 W and rows of up to 17 elements gain nothing.  Alone / two / four, whole step, us:
  // 128x128x64x33, r 16,8 behind 32,32 185.5 / 184.2 / -; 100x100x64x65, r 16,8 217 / 212 / 207; 128x128x128x33, r 16,8, bf16 G 296 /
  // 299 / 284; 50x50x64x65 73.3 / 71.0 / 69.5; 128x128x128x65, r 32,16 741 / 725 / 732; 64x64x128x65, r 32,16 207 / 201 / 200;
  // 100x100x96x40, r 30,6 221 / 217 / -; but 64x64x64x33, r 30,16 80.9 / 85.3 / -; 100x100x64x17, r 8,4 67.5 / 68.2 / -; 128x128x64x65,
  // bf16 G and W 190.6 / 189.5 / 190.8.
  // Where a workgroup then has fewer slabs than one of k_head, it takes them on the same XCD: the support's places and values that one
  // of the kernels has written or read lie in the other's L2.  Alone / two, each on the next XCD / two, 1, 5 and 30 % in the
  // support: 2106 slabs of 44x29, r 8,8, 30 % 45.1 / 46.8 / 44.5; 1600 of 64x33, r 16,8 35.6 / 35.3 / 34.7, 35.8 / 36.0 / 35.0 and
  // 45.5 / 46.3 / 43.9; 2700 of 115x19, r 30,7 61.9 / 61.9 / 60.9, 62.4 / 63.2 / 61.5 and 79.3 / 76.5 / 76.1; where gs outgrows the
  // L2s nothing changes.
  // Slabs of two tiles are not shared from 2560 on to 3072 (a round of 2048 wavefronts and a part: with two for a slab two rounds and as
  // large a part; alone / two: 2700 of 44x29, r 8,8 37.4 / 38.5, of 64x33, r 16,16 57.3 / 58.5, of 39x19, r 8,4 31.0 / 31.5; but 2401 of 44x22,
  // r 11,12 39.7 / 37.5, 2100 of 39x19, r 16,11 37.3 / 35.6, 3540 of 64x33, r 16,16 68.1 / 65.0), nor from there on if the second has less than 12 rows of 32
  // for its wavefront (16000 of 39x19, r 16,11 117.1 / 121.0, 30 % 136.9 / 149.6; 8010 74.7 / 76.6; but 5593 of 45x29, r 13,14 79.5 / 78.0,
  // 9401 of 54x28, r 6,11 94.5 / 92.1).  Nor, for ranks of 17 and more in mode N-1, 1280 to 2047 slabs, one for each wavefront (1600 of
  // 126x27, r 30,8 52.1 / 54.0, of 115x19, r 30,7 43.1 / 43.8; but 1122 of 126x27 47.5 / 44.8, 2100 70.2 / 64.3).
  const int many = K2 <= 16 ? (S % 4 == 0 ? 4 : 2) : S >= 6 || (K <= 8 && S >= 4) ? 2 : 1;
  const bool levels = S == 2 ? nslabs < 5 * kWholeSlabs / 2 || (nslabs >= 3 * kWholeSlabs && 8 * (I2 - R) >= 3 * R)
                             : K2 <= 16 || nslabs < 5 * kWholeSlabs / 4 || nslabs >= 2 * kWholeSlabs;
  const int together = !split && levels && tail_shares(wdtype, columns_class(M)) && S % many == 0 ? many : 1;
  const int64_t units = split ? nslabs * S : nslabs * together;
  const int full = tail_lds(4, M, I2, K2, K) <= kLdsLimit / 2 ? 4 : tail_lds(8, M, I2, K2, K) <= kLdsLimit ? 8 : 4;
  // Few tiles: a wavefront each.  Where coefficients go to LDS (tail_coef_lds) it then takes its operands straight into
  // registers; while all such tiles are resident that is the faster one for up to 8 columns of rank, beyond that up to
  // three per compute unit.  Us, those / LDS / float32 operands as before: 42x42x44, r 13,14 5.8 / 7.4 / 6.9; 108x58x67, r 17,16 8.0 /
  // 10.7 / 10.0; 380 slabs of 86x61, r 19,5 11.0 / 13.9 / 14.4; 552 of 82x54, r 22,8 14.3 / 13.6 / 16.1; 324 of 65x58, r 21,14
  // 12.9 / 11.4 / 15.0.
  const bool in_lds = tail_coef_lds(columns_class(M), K <= 8 ? 1 : 2);
  const bool one = in_lds && split && units <= (K <= 8 ? 3 * kWholeSlabs : 768);
  const int W = !one && (in_lds || units >= kWholeSlabs) ? full : 1;
  const size_t lds = tail_lds(W, M, I2, K2, K, one);
  TailArgs a{y1, U2, U3, w, K, M, I2, K2, S, (int)nslabs, split ? 1 : W % together || together == 1 ? 0 : together, decay, c_alpha};
  const SparseAdam sp = sparse_adam(omega, tile_start, gs, ms, vs, beta1, beta2, inv_c1, inv_c2, eps, c_lambda, 0);
  const int ct = columns_class(M), nc = K <= 8 ? 1 : 2, sa = step_class(K2);
#define TGRAD_TAIL(WD_, T_, C_, A_)                                                                          \
  do {                                                                                                       \
    if constexpr (tail_coef_lds(T_, C_)) {                                                                   \
      if (one) {                                                                                             \
        k_tail<WD_, T_, C_, A_, true><<<dim3((unsigned)units), dim3(64), lds, s>>>(a, sp);                   \
        break;                                                                                               \
      }                                                                                                      \
    }                                                                                                        \
    allow_lds(k_tail<WD_, T_, C_, A_, false>, lds);                                                          \
    const unsigned grid = end_grid(k_tail<WD_, T_, C_, A_, false>, W, lds, units);                           \
    k_tail<WD_, T_, C_, A_, false><<<dim3(grid), dim3(64 * W), lds, s>>>(a, sp);                             \
  } while (0)
#define TGRAD_TAIL_A(WD_, T_, C_)                                                                            \
  do {                                                                                                       \
    if (sa == 2) TGRAD_TAIL(WD_, T_, C_, 2); else if (sa == 4) TGRAD_TAIL(WD_, T_, C_, 4); else TGRAD_TAIL(WD_, T_, C_, 8); \
  } while (0)
#define TGRAD_TAIL_T(WD_)                                                                                    \
  do {                                                                                                       \
    if (ct == 2) { if (nc == 1) TGRAD_TAIL_A(WD_, 2, 1); else TGRAD_TAIL_A(WD_, 2, 2); }                     \
    else if (ct == 3) { if (nc == 1) TGRAD_TAIL_A(WD_, 3, 1); else TGRAD_TAIL_A(WD_, 3, 2); }                \
    else if (ct == 4) { if (nc == 1) TGRAD_TAIL_A(WD_, 4, 1); else TGRAD_TAIL_A(WD_, 4, 2); }                \
    else { if (nc == 1) TGRAD_TAIL_A(WD_, 9, 1); else TGRAD_TAIL_A(WD_, 9, 2); }                             \
  } while (0)
  if (wdtype == TGRAD_C64) TGRAD_TAIL_T(TGRAD_C64); else TGRAD_TAIL_T(TGRAD_CBF16);
#undef TGRAD_TAIL_T
#undef TGRAD_TAIL_A
#undef TGRAD_TAIL
}

}  // namespace tgrad
