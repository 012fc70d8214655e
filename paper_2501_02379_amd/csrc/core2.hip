// k_core2: everything between the first compression stages and the last reconstruction stages once two
// modes (the two leading ones) are left: y is (I0, I1, Cc), its Cc complex columns contiguous.  Every
// column c goes through
//   g_L[m0, m1, c] = sum_{i0, i1} conj(U0[i0, m0]) conj(U1[i1, m1]) y[i0, i1, c]   last two compression stages
//   N_L            = AdamUpdate(g_L)                (appendix algorithm "Adam with low-rank tensor decomposition")
//   z[i0, i1, c]   = sum_{m0, m1} U0[i0, m0] U1[i1, m1] N_L[m0, m1, c]             first two reconstruction stages
// on its own, so a workgroup that owns a column runs the whole chain between workgroup barriers: nothing
// travels through memory between the five steps, and the launches, prologues and tails of three kernels
// become one.  What it pays for that: a workgroup reads 8 bytes of every cache line of y (neighbouring columns
// belong to other workgroups), so it is the kernel of small leading modes, where launches cost more than
// lines (core2_kernel_fits has the line and both sides of it).
//
// Tiles are 16 x 16 (v_mfma_f32_16x16x4f32, the same rate as 32x32x2), one for both ranks; a wavefront has one tile of 16
// rows i0 at a time.  Operand layout (64 lanes, g = lane / 16, c = lane % 16):
//   A[i = c][k = g],  B[k = g][j = c],  D register r: D[i = 4 g + r][j = c].
// The accumulator layout of one stage is the operand layout of the next - register r of D holds the
// rows 4 g + r over the four lane groups, and a matrix-core step contracts exactly four rows, one per
// group - so no stage transposes anything:
//   1  T[i0, m1]   = sum_i1 y[i0, i1] conj(U1[i1, m1])   A = y (lane = row i0), B = U1 (LDS);  D: i0 in registers
//   2  P[m0, m1]   = sum_i0 conj(U0[i0, m0]) T[i0, m1]   A = U0, B = T straight from the accumulators; the
//                                                        wavefronts' partial sums meet in LDS, fixed order
//   -  AdamUpdate on the workgroup's core entries, N_L back into LDS in accumulator layout
//   3  R[m1, i0]   = sum_m0 N_L[m0, m1] U0[i0, m0]       A = N_L (LDS), B = U0;  D: m1 in registers, i0 in lanes
//   4  z[i0, i1]   = sum_m1 R[m1, i0] U1[i1, m1]         A = R straight from the accumulators, B = U1 (LDS)
// With fewer than 8 row tiles the spare wavefronts take slices of i1 of the same rows: stage 2 is linear,
// so partial T's go straight into the partial P's that are summed anyway; in stage 4 the wavefronts of
// a row tile deal its column tiles among themselves (stage 3 is then computed once per wavefront).
#include "device_common.h"
#include "launch_util.h"

namespace tgrad {

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kBatch = 8;                    // steps of y per lane in flight (twice that while a batch is computed)

struct Core2Args {
  const float* y;       // (I0, I1, Cc) complex
  float* z;             // the same shape; may be y (a workgroup writes only the column it alone has read, after its
                        // last read)
  const float2* U0;     // (I0, M0)
  const float2* U1;     // (I1, M1)
  int I0, I1, M0, M1;
  int Cc;
};

struct Core2Adam {
  float2* m;            // first moments, (M0, M1, Cc) complex
  float* v;             // second moments
  float2* g_out;        // compressed gradient, written for the state accessors
  float beta1, beta2, inv_c1, inv_c2, eps;
};

constexpr int kSlot = 2 * 4 * 64;            // floats of a wavefront's partial P in LDS: [comp][r][lane]

__global__ __launch_bounds__(kThreads) void k_core2(Core2Args a, Core2Adam ad) {
  extern __shared__ float2 sL[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  // neighbouring columns share cache lines of y: consecutive columns go to workgroups 8 apart, i.e. to the
  // same XCD (one L2) under round-robin dispatch
  const int per = (int)gridDim.x >> 3;        // the grid is a multiple of 8 (host)
  const int plane = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
  if (plane >= a.Cc) return;
  const int I0 = a.I0, I1 = a.I1, M0 = a.M0, M1 = a.M1;
  const int J1 = (I1 + 3) >> 2;               // steps of stage 1
  const int Q1 = (I1 + 15) >> 4;              // column tiles of stage 4
  const int RT = (I0 + 15) >> 4;              // row tiles
  const int nsl = RT >= kWaves ? 1 : kWaves / RT;      // wavefronts per row tile
  const int slice = RT >= kWaves ? 0 : wave / RT;
  const int t_first = RT >= kWaves ? wave : wave - slice * RT;
  const bool active = slice < nsl && t_first < RT;     // (wave-uniform) idle wavefronts only pass the barriers
  const int64_t row = (int64_t)a.Cc * 2;      // floats between consecutive i1 of y
  const int64_t slab = row * I1;              // floats between consecutive i0 of y
  // LDS: the partial sums of the eight wavefronts ([wave][comp][r][lane] floats; N_L in the first), the stage-1 operands
  // [J1][64], the stage-4 operands [Q1][4][64], each in a place of its own: three barriers are enough
  // (with the sums in two rounds in the place of the operands there were six; static step 32x32x12x7 21.2 us, now 20.7)
  const int nA = J1 * 64;
  float* red = reinterpret_cast<float*>(sL);
  float2* sT1 = sL + kWaves * kSlot / 2;
  const int nB = Q1 * 4 * 64;

  // ---- prologue: the first rows of y, then all operands go in flight ----
  const int j_per = (J1 + nsl - 1) / nsl;
  const int j0 = slice * j_per, j1 = j0 + j_per < J1 ? j0 + j_per : J1;
  const float* yp = a.y + (int64_t)plane * 2;
  auto load_y = [&](const float* rowp, int j) -> float2 {
    const int i1 = 4 * j + grp;
    return *reinterpret_cast<const float2*>(rowp + (int64_t)(i1 < I1 ? i1 : I1 - 1) * row);
  };
  auto row_ptr = [&](int t) -> const float* {
    const int i0 = 16 * t + col;
    return yp + (int64_t)(i0 < I0 ? i0 : I0 - 1) * slab;
  };
  float2 cur[kBatch];
  if (active) {
    const float* rp = row_ptr(t_first);
#pragma unroll
    for (int u = 0; u < kBatch; ++u) cur[u] = load_y(rp, j0 + u);
  }
  // moments of this thread's core entry (register tid / 64 of lane tid % 64; the upper four wavefronts have none)
  const int em0 = 4 * grp + (wave & 3);
  const bool live = wave < 4 && em0 < M0 && col < M1;
  const int64_t cidx = live ? ((int64_t)em0 * M1 + col) * a.Cc + plane : 0;
  const float2 mm = ad.m[cidx];
  const float vv = ad.v[cidx];
  // (sizes made scalar: a product that the compiler keeps in a vector register turns every load into a loop over the lanes)
  const FactorRef fU0 = factor_ref(a.U0, __builtin_amdgcn_readfirstlane(I0 * M0));
  const FactorRef fU1 = factor_ref(a.U1, __builtin_amdgcn_readfirstlane(I1 * M1));
  auto u1_at = [&](int i1, int m1) -> float2 { return factor_entry(fU1, i1, m1, M1, i1 < I1 && m1 < M1); };
  auto u0_at = [&](int i0, int m0) -> float2 { return factor_entry(fU0, i0, m0, M0, i0 < I0 && m0 < M0); };
  // the U0 operands of stage 2 (f2) and of stage 3 (f3) of the first row tile are requested here as well: asked for
  // where they are used, each is a memory round trip in front of its stage (16x16x8x5: 10.2 us, now 8.2)
  float2 f2[4], f3[4];
  auto fetch_f2 = [&](int t) {                                // U0[16 t + 4 g + r][c]
#pragma unroll
    for (int r = 0; r < 4; ++r) f2[r] = u0_at(16 * t + 4 * grp + r, col);
  };
  auto fetch_f3 = [&](int t) {                                // U0[16 t + c][4 g + r]
#pragma unroll
    for (int r = 0; r < 4; ++r) f3[r] = u0_at(16 * t + col, 4 * grp + r);
  };
  if (active) {
    fetch_f2(t_first);
    fetch_f3(t_first);
  }
  // both tables in one go, behind those requests: staged one after the other they were two memory round trips
  stage_table(sT1, nA + nB, tid, kThreads, [&](int e) -> float2 {            // U1[4 j + g][c], then U1[16 q + c][4 g + r]
    const int l = e & 63, n = (e >> 6) - J1, r = n & 3, q = n >> 2;
    const bool first = n < 0;
    return u1_at(first ? 4 * (n + J1) + (l >> 4) : 16 * q + (l & 15), first ? l & 15 : 4 * (l >> 4) + r);
  });
  __syncthreads();

  // ---- stages 1 and 2 over this wavefront's row tiles ----
  v4f p[2];
  p[0] = p[1] = (v4f){0.f, 0.f, 0.f, 0.f};
  if (active) {
    for (int t = t_first; t < RT; t += kWaves) {
      const float* rp = row_ptr(t);
      if (t != t_first) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) cur[u] = load_y(rp, j0 + u);
        fetch_f2(t);
      }
      v4f tt[2];
      tt[0] = tt[1] = (v4f){0.f, 0.f, 0.f, 0.f};
      auto stage1 = [&](float2 v, int j) {
        const float2 f = sT1[j * 64 + lane];
        tt[0] = mfma16(v.x, f.x, tt[0]);                       // re: yr ur + yi ui;  im: yi ur - yr ui
        tt[1] = mfma16(v.y, f.x, tt[1]);
        tt[0] = mfma16(v.y, f.y, tt[0]);
        tt[1] = mfma16(v.x, -f.y, tt[1]);
      };
      int j = j0;
      for (; j + kBatch <= j1; j += kBatch) {
        float2 nxt[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) nxt[u] = load_y(rp, j + kBatch + u);
        __builtin_amdgcn_sched_barrier(0);                    // the loads stay in front of the batch they overlap
#pragma unroll
        for (int u = 0; u < kBatch; ++u) stage1(cur[u], j + u);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) cur[u] = nxt[u];
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        if (j + u < j1) stage1(cur[u], j + u);
#pragma unroll
      for (int r = 0; r < 4; ++r) {                            // re: ur tr + ui ti;  im: ur ti - ui tr
        const float2 f = f2[r];
        p[0] = mfma16(f.x, tt[0][r], p[0]);
        p[1] = mfma16(f.x, tt[1][r], p[1]);
        p[0] = mfma16(f.y, tt[1][r], p[0]);
        p[1] = mfma16(-f.y, tt[0][r], p[1]);
      }
    }
  }
  // ---- the wavefronts' partial sums, always added in the same order ----
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave * kSlot + (i * 4 + r) * 64 + lane] = p[i][r];
  __syncthreads();
  // ---- AdamUpdate; N_L replaces the partial sums of slot 0 (each entry is read and written by one thread) ----
  if (wave < 4) {
    float* pr = red + wave * 64 + lane;
    float* pi = pr + 256;
    float gre = 0.f, gim = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      gre += pr[w * kSlot];
      gim += pi[w * kSlot];
    }
    float2 m = mm;
    m.x = ad.beta1 * m.x + (1.f - ad.beta1) * gre;
    m.y = ad.beta1 * m.y + (1.f - ad.beta1) * gim;
    const float v = ad.beta2 * vv + (1.f - ad.beta2) * (gre * gre + gim * gim);
    const float d = 1.f / (sqrtf(v * ad.inv_c2) + ad.eps);
    float nr = 0.f, ni = 0.f;
    if (live) {
      ad.m[cidx] = m;
      ad.v[cidx] = v;
      ad.g_out[cidx] = make_float2(gre, gim);
      nr = m.x * ad.inv_c1 * d;
      ni = m.y * ad.inv_c1 * d;
    }
    *pr = nr;
    *pi = ni;
  }
  __syncthreads();
  if (!active) return;                                         // no barrier follows
  // ---- stages 3 and 4 ----
  float* zp = a.z + 2 * (int64_t)plane;
  for (int t = t_first; t < RT; t += kWaves) {
    v4f rr[2];
    rr[0] = rr[1] = (v4f){0.f, 0.f, 0.f, 0.f};
    if (t != t_first) fetch_f3(t);
#pragma unroll
    for (int r = 0; r < 4; ++r) {                              // re: nr ur - ni ui;  im: ni ur + nr ui
      const float2 f = f3[r];
      const float nr = red[r * 64 + lane], ni = red[(4 + r) * 64 + lane];
      rr[0] = mfma16(nr, f.x, rr[0]);
      rr[1] = mfma16(ni, f.x, rr[1]);
      rr[0] = mfma16(ni, -f.y, rr[0]);
      rr[1] = mfma16(nr, f.y, rr[1]);
    }
    for (int q = slice; q < Q1; q += nsl) {
      v4f z[2];
      z[0] = z[1] = (v4f){0.f, 0.f, 0.f, 0.f};
      const float2* ft = sT1 + nA + q * 256 + lane;
#pragma unroll
      for (int r = 0; r < 4; ++r) {                            // re: rr ur - ri ui;  im: rr ui + ri ur
        const float2 f = ft[r * 64];
        z[0] = mfma16(rr[0][r], f.x, z[0]);
        z[1] = mfma16(rr[0][r], f.y, z[1]);
        z[0] = mfma16(rr[1][r], -f.y, z[0]);
        z[1] = mfma16(rr[1][r], f.x, z[1]);
      }
      const int i1 = 16 * q + col;
      if (i1 < I1) {
        float* zt = zp + (int64_t)(16 * t + 4 * grp) * slab + (int64_t)i1 * row;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (16 * t + 4 * grp + r < I0)
            *reinterpret_cast<float2*>(zt + (int64_t)r * slab) = make_float2(z[0][r], z[1][r]);
      }
    }
  }
}

size_t core2_lds(int I1) {
  return (size_t)kWaves * kSlot * 4 + (size_t)((I1 + 3) / 4) * 64 * 8 + (size_t)((I1 + 15) / 16) * 4 * 64 * 8;
}

}  // namespace

// Where the two leading modes (extents I0, I1, ranks M0, M1) and the Cc columns of the core between them are one launch.
// Against the three kernels k_mid, k_core, k_expand, difference of a whole step of 17 ... 45 us (one launch - three):
//   at 8, 64, 128, 256 columns (and 512, 2048) with ranks a quarter of the extents
//     8x8 -5, -4, -3, -3 (-1, +22); 16x16 -5, -4, -3, -3 (+1, +25); 32x32 -2, -1, -1, -2 (+4, +30); 40x40 -2, -2, -2, -1 (0, +23);
//   at 8, 64, 128, 256 columns with ranks 8, 8
//     8x200 -4, -3, -3, -1; 100x16 -4, -3, -4, -2; 16x64 -4, -2, -1, +1; 32x50 -2, -1, 0, +1;
//   ... with ranks 16, 16
//     32x32 -2, -1, 0, 0; 40x40 -2, 0, 0, 0; 16x64 -2, -1, 0, +1; 16x100 -2, 0, +1, +3;
//   ... of larger modes
//     46x46 (r 23,23) +2, +3, +4, +1; 64x64 (r 16,16) +3, +3, +5, +4; 128x40 (r 32,10) +1, +4, +3, +5;
//     128x128 (r 32,32) +22, +22, +20, +17, and +36 with 384 columns.
// So: up to 40 x 40 with ranks of one tile and up to one workgroup per compute unit the saved launches win; after that the
// whole cache lines of the three kernels do.
bool core2_kernel_fits(int I0, int I1, int M0, int M1, int64_t Cc) {
  return I0 * I1 <= 1600 && M0 <= 16 && M1 <= 16 && Cc >= 1 && Cc <= 256;
}

void launch_core2(hipStream_t s, const float2* x, const float2* U0, const float2* U1, int I0, int I1, int M0, int M1,
                  int64_t Cc, float2* m, float* v, float2* g_out, float beta1, float beta2, float inv_c1, float inv_c2,
                  float eps, float2* z) {
  if (Cc <= 0) return;
  const size_t lds = core2_lds(I1);
  Core2Args a{reinterpret_cast<const float*>(x), reinterpret_cast<float*>(z), U0, U1, I0, I1, M0, M1, (int)Cc};
  Core2Adam ad{m, v, g_out, beta1, beta2, inv_c1, inv_c2, eps};
  allow_lds(k_core2, lds);
  k_core2<<<dim3((unsigned)((Cc + 7) / 8 * 8)), dim3(kThreads), lds, s>>>(a, ad);
}

}  // namespace tgrad
