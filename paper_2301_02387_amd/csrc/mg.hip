// Geometric multigrid preconditioner for the pair Poisson solves: a V-cycle
// per instance over the hierarchy built by build_multigrid (the operator's own
// Q_p space, Q2 below Q3 and Q1 on the same leaves, Q1 on shallower refinements,
// coarser base grids, a dense inverse at the bottom), with Chebyshev smoothing
// preconditioned by the diagonal.  All n^2 real pair columns go through every
// pass together ([rows][ncol] arrays), and every pass covers all instances of
// a batch in one launch: blockIdx.y selects the instance's level record, and
// records of levels an instance does not have are inactive.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "devutil.hpp"
#include "kernels.hpp"
#include "mg.hpp"

namespace mh {

#define INSTANCE const DevMesh& d = dm[blockIdx.y]

// sum of val[t] x[col[t] ncol + c] over t = beg, beg + stride, ... < end, for end > beg.  Rounds of 8 entries:
// the indices and coefficients of the next round are requested before this
// round's gathers, so each round waits for one memory latency.  Entries past
// the end repeat the last one with coefficient 0 (in-bounds loads, no branch).
template <class IP, class DP, class XP>
__device__ __forceinline__ double row_gather_dot(IP col, DP val, int beg, int end, int stride, XP x, int ncol, int c) {
  double s = 0.0;
  int jn[8];
  double an[8];
#pragma unroll
  for (int h = 0; h < 8; ++h) {
    const int tt = beg + h * stride;
    const int tc = tt < end ? tt : end - 1;
    jn[h] = col[tc];
    an[h] = tt < end ? val[tc] : 0.0;
  }
  for (int t = beg; t < end; t += 8 * stride) {
    int jc[8];
    double ac[8];
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      jc[h] = jn[h];
      ac[h] = an[h];
    }
    if (t + 8 * stride < end) {
#pragma unroll
      for (int h = 0; h < 8; ++h) {
        const int tt = t + (8 + h) * stride;
        const int tc = tt < end ? tt : end - 1;
        jn[h] = col[tc];
        an[h] = tt < end ? val[tc] : 0.0;
      }
    }
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      const int64_t j = (int64_t)jc[h] * ncol + c;
      s += ac[h] * (double)x[j];
    }
  }
  return s;
}

// The same with V adjacent columns per lane (c0 .. c0 + V, 16-byte loads;
// ncol and c0 multiples of V): s[v] += the entries' sum for column c0 + v.
template <int V, class IP, class DP, class XP>
__device__ __forceinline__ void row_gather_v(IP col, DP val, int beg, int end, int stride, XP x, int ncol, int c0,
                                             double* s) {
  int jn[8];
  double an[8];
#pragma unroll
  for (int h = 0; h < 8; ++h) {
    const int tt = beg + h * stride;
    const int tc = tt < end ? tt : end - 1;
    jn[h] = col[tc];
    an[h] = tt < end ? val[tc] : 0.0;
  }
  for (int t = beg; t < end; t += 8 * stride) {
    int jc[8];
    double ac[8];
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      jc[h] = jn[h];
      ac[h] = an[h];
    }
    if (t + 8 * stride < end) {
#pragma unroll
      for (int h = 0; h < 8; ++h) {
        const int tt = t + (8 + h) * stride;
        const int tc = tt < end ? tt : end - 1;
        jn[h] = col[tc];
        an[h] = tt < end ? val[tc] : 0.0;
      }
    }
    double xv[8][V];
#pragma unroll
    for (int h = 0; h < 8; ++h) load_vals<V>(x + (int64_t)jc[h] * ncol + c0, xv[h]);
#pragma unroll
    for (int h = 0; h < 8; ++h)
#pragma unroll
      for (int v = 0; v < V; ++v) s[v] += ac[h] * xv[h][v];
  }
}

// coarse.r = R fine.t (t: the residual r - A z) for each instance whose fine
// record is active.  A restriction row gathers every fine node in the support
// of a coarse basis function, so G lanes take a row: groups of cw lanes (a power
// of two >= ncol) split its entries, lane c of a group holds column c, and the
// groups are combined by shuffles; rows swept by XCD.
__global__ void __launch_bounds__(NT) k_mg_restrict(const MgLevelDev* __restrict__ fine,
                                                    const MgLevelDev* __restrict__ coarse, int ncol, int cw, int G) {
  const MgLevelDev& F = fine[blockIdx.y];
  if (!F.active || (F.done && *F.done)) return;
  const MgLevelDev& C = coarse[blockIdx.y];
  const auto* ptr = gbl(F.r_ptr);
  const auto* col = gbl(F.r_col);
  const auto* val = gbl(F.r_val);
  const auto* t = gbl((const double*)F.t);
  const auto* tf = gbl((const float*)F.tf);
  const bool f32 = F.f32 != 0;
  auto* y = gblw(C.r);
  const int lane = threadIdx.x & (G - 1);
  const int grp = lane / cw, c = lane - grp * cw, ngrp = G / cw;
  const XcdSweep sw = xcd_sweep(C.N, NT / G);
  for (int64_t w = sw.start + threadIdx.x / G; w < sw.end; w += sw.step) {
    double s = 0.0;
    if (c < ncol) {
      const int beg = ptr[w] + grp, end = ptr[w + 1];
      if (end > beg)
        s = f32 ? row_gather_dot(col, val, beg, end, ngrp, tf, ncol, c)
                : row_gather_dot(col, val, beg, end, ngrp, t, ncol, c);
    }
    for (int off = G / 2; off >= cw; off >>= 1) s += __shfl_xor(s, off, 64);
    if (grp == 0 && c < ncol) y[w * ncol + c] = s;
  }
}

// The restriction with V columns per lane (ncol a multiple of V, cw a power
// of two >= ncol / V lanes per group): 64 / cw groups split a row's entries,
// each with eight entries in flight.
template <int V>
__global__ void __launch_bounds__(NT) k_mg_restrict_v(const MgLevelDev* __restrict__ fine,
                                                      const MgLevelDev* __restrict__ coarse, int ncol, int cw) {
  const MgLevelDev& F = fine[blockIdx.y];
  if (!F.active || (F.done && *F.done)) return;
  const MgLevelDev& C = coarse[blockIdx.y];
  const auto* ptr = gbl(F.r_ptr);
  const auto* col = gbl(F.r_col);
  const auto* val = gbl(F.r_val);
  const auto* t = gbl((const double*)F.t);
  const auto* tf = gbl((const float*)F.tf);
  const bool f32 = F.f32 != 0;
  auto* y = gblw(C.r);
  const int lane = threadIdx.x & 63;
  const int grp = lane / cw, c0 = (lane - grp * cw) * V, ngrp = 64 / cw;
  const bool act = c0 < ncol;
  const XcdSweep sw = xcd_sweep(C.N, NT / 64);
  for (int64_t w = sw.start + (threadIdx.x >> 6); w < sw.end; w += sw.step) {
    double s[V];
#pragma unroll
    for (int v = 0; v < V; ++v) s[v] = 0.0;
    const int beg = ptr[w] + grp, end = ptr[w + 1];
    if (act && end > beg) {
      if (f32) row_gather_v<V>(col, val, beg, end, ngrp, tf, ncol, c0, s);
      else row_gather_v<V>(col, val, beg, end, ngrp, t, ncol, c0, s);
    }
    for (int off = 32; off >= cw; off >>= 1)
#pragma unroll
      for (int v = 0; v < V; ++v) s[v] += __shfl_xor(s[v], off, 64);
    if (grp == 0 && act)
#pragma unroll
      for (int v = 0; v < V; ++v) y[w * ncol + c0 + v] = s[v];
  }
}

// fine.z += P coarse.z with V columns per lane and L lanes per row (a power
// of two >= ncol / V), so a wave takes 64 / L rows at once; rows swept by XCD.
template <int V, int L>
__global__ void __launch_bounds__(NT) k_mg_prolong_v(const MgLevelDev* __restrict__ fine,
                                                     const MgLevelDev* __restrict__ coarse, int ncol) {
  const MgLevelDev& F = fine[blockIdx.y];
  if (!F.active || (F.done && *F.done)) return;
  const MgLevelDev& C = coarse[blockIdx.y];
  const auto* ptr = gbl(F.p_ptr);
  const auto* col = gbl(F.p_col);
  const auto* val = gbl(F.p_val);
  const auto* x = gbl((const double*)C.z);
  auto* z = gblw(F.z);
  auto* zf = gblw(F.zf);
  const bool f32 = F.f32 != 0;
  const int c0 = (int)(threadIdx.x & (L - 1)) * V;
  const bool act = c0 < ncol;
  const XcdSweep sw = xcd_sweep(F.N, NT / L);
  for (int64_t i = sw.start + threadIdx.x / L; i < sw.end; i += sw.step) {
    const int beg = ptr[i], end = ptr[i + 1];
    if (!act || end <= beg) continue;
    double s[V];
#pragma unroll
    for (int v = 0; v < V; ++v) s[v] = 0.0;
    row_gather_v<V>(col, val, beg, end, 1, x, ncol, c0, s);
    const int64_t e = i * ncol + c0;
    double zo[V];
    if (f32) {
      load_vals<V>(zf + e, zo);
#pragma unroll
      for (int v = 0; v < V; ++v) zf[e + v] = (float)(zo[v] + s[v]);
    } else {
      load_vals<V>(z + e, zo);
#pragma unroll
      for (int v = 0; v < V; ++v) z[e + v] = zo[v] + s[v];
    }
  }
}

// fine.z += P coarse.z for each instance whose fine record is active
__global__ void __launch_bounds__(NT) k_mg_prolong(const MgLevelDev* __restrict__ fine,
                                                   const MgLevelDev* __restrict__ coarse, int ncol) {
  const MgLevelDev& F = fine[blockIdx.y];
  if (!F.active || (F.done && *F.done)) return;
  const MgLevelDev& C = coarse[blockIdx.y];
  const int64_t total = F.N * ncol;
  const auto* ptr = gbl(F.p_ptr);
  const auto* col = gbl(F.p_col);
  const auto* val = gbl(F.p_val);
  const auto* x = gbl((const double*)C.z);
  auto* z = gblw(F.z);
  auto* zf = gblw(F.zf);
  const bool f32 = F.f32 != 0;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < total; e += (int64_t)gridDim.x * NT) {
    const int64_t i = e / ncol;
    const int c = (int)(e - i * ncol);
    const int beg = ptr[i], end = ptr[i + 1];
    if (end > beg) {
      const double v = row_gather_dot(col, val, beg, end, 1, x, ncol, c);
      if (f32) zf[e] = (float)((double)zf[e] + v);
      else z[e] += v;
    }
  }
}

// z = Ainv r on each instance's coarsest level (dense, symmetric), on the FP64
// matrix cores: a workgroup of sixteen waves takes 16 rows and all columns (NCT
// tiles of 16), each wave a sixteenth of the contraction; the partial tiles are
// added in LDS.  The pass is bound by reading Ainv, which is read once for all
// columns.  As Ainv is symmetric, rows i0 .. i0 + 15 of a contraction index j
// are taken from its row j, 128 consecutive bytes (lane layout of
// k_moments_mfma).  Measured, against a wave per row and 8 columns that read
// Ainv again for every 8: 1154 -> 54 us at 4,096 unknowns x 36 columns
// (670 MB -> 134 MB read), 15.8 -> 14.6 us at 1,979 x 4
constexpr int MC_W = 16;   // waves of a workgroup
template <int NCT>
__global__ void __launch_bounds__(64 * MC_W) k_mg_coarse(const MgLevelDev* __restrict__ co, int ncol) {
  const MgLevelDev& L = co[blockIdx.y];
  const int64_t n = L.N;
  const int64_t i0 = (int64_t)blockIdx.x * 16;
  if (i0 >= n || (L.done && *L.done)) return;
  __shared__ double lds[MC_W][256];
  typedef double dvec4c_t __attribute__((ext_vector_type(4)));
  const auto* Ainv = gbl(L.cinv);
  const auto* r = gbl((const double*)L.r);
  auto* z = gblw(L.z);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int64_t ia = i0 + li < n ? i0 + li : n - 1;   // rows past the end are computed and not stored
  // this wave's contraction range, in steps of 4
  const int64_t steps = (n + 3) / 4, per = (steps + MC_W - 1) / MC_W;
  const int64_t s0 = wave * per, s1 = s0 + per < steps ? s0 + per : steps;
  dvec4c_t acc[NCT];
#pragma unroll
  for (int u = 0; u < NCT; ++u) acc[u] = dvec4c_t{0.0, 0.0, 0.0, 0.0};
  constexpr int U = NCT <= 2 ? 8 : 4;   // steps whose loads are in flight together
  for (int64_t st = s0; st < s1; st += U) {
    double av[U], bv[U][NCT];
#pragma unroll
    for (int h = 0; h < U; ++h) {
      const int64_t j = 4 * (st + h) + lk;
      const bool ok = st + h < s1 && j < n;
      const int64_t jc = ok ? j : n - 1;   // in-bounds load, weight zero
      const double a = Ainv[jc * n + ia];
      av[h] = ok ? a : 0.0;
#pragma unroll
      for (int u = 0; u < NCT; ++u) {
        const int c = 16 * u + li;
        const double b = r[jc * ncol + (c < ncol ? c : 0)];
        bv[h][u] = c < ncol ? b : 0.0;
      }
    }
#pragma unroll
    for (int h = 0; h < U; ++h)
#pragma unroll
      for (int u = 0; u < NCT; ++u) acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[h], bv[h][u], acc[u], 0, 0, 0);
  }
#pragma unroll
  for (int u = 0; u < NCT; ++u) {
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) lds[wave][(4 * v + lk) * 16 + li] = acc[u][v];
    __syncthreads();
    if (threadIdx.x < 256) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < MC_W; ++w) t += lds[w][threadIdx.x];
      const int64_t i = i0 + (threadIdx.x >> 4);
      const int c = 16 * u + (int)(threadIdx.x & 15);
      if (i < n && c < ncol) z[i * ncol + c] = t;
    }
  }
}

static dim3 level_grid(int64_t n, int ncol, int ni) { return dim3(nblocks(n * ncol, NT, 16384), ni); }

// Coarse-level passes with the operator product fused in, LN lanes per row
// and V adjacent columns per lane (16-byte loads for V = 4).  The smoothing is
// Chebyshev of degree 2 (zin and zout are the level's z and t arrays, so the
// rows gathered are never the rows written):
//  - LP_ZERO, both steps from zero: the first step's c0 D^-1 r is formed in the
//    product (a_vd holds the values times D^-1 of their columns), r -> z;
//  - LP_STEP0, LP_STEP1, the two steps on a given correction: z -> t with d kept,
//    then t -> z;
//  - LP_RES, the residual t = r - A z that the restriction reads.
// Bound by the gathers (13 rows of 512 B per row at 64 columns, out of L2) on
// large levels, by the index -> gather chain of the longest rows on small ones.
// Per cycle, five passes before -> four: Q2 level of H2O (429,000 rows x 64
// columns) 1607 -> 1428 us, of H2 (18,700 x 4) 50.5 -> 28.9 us.  Rows swept in
// one range per XCD: 1442 us, and 54.9 us at H2 (long rows lie together).
enum { LP_ZERO = 0, LP_STEP0 = 1, LP_STEP1 = 2, LP_RES = 3 };
template <int MODE, int V, int LN>
__global__ void __launch_bounds__(NT) k_mg_level_pass(const MgLevelDev* __restrict__ lv, int ncol, int cw) {
  const MgLevelDev& L = lv[blockIdx.y];
  if (!L.active || (L.done && *L.done)) return;
  const double b = L.lmax, a = L.lmax / MG_RANGE;
  const double theta = 0.5 * (b + a), delta = 0.5 * (b - a), sigma = theta / delta;
  const double c0 = 1.0 / theta, rn = 1.0 / (2.0 * sigma - 1.0 / sigma);
  const double c1 = rn / sigma, c2 = 2.0 * rn / delta;
  const auto* ptr = gbl(L.a_ptr);
  const auto* col = gbl(L.a_col);
  const auto* val = gbl(MODE == LP_ZERO ? L.a_vd : L.a_val);
  const auto* dinv = gbl(L.dinv);
  const auto* r = gbl((const double*)L.r);
  const auto* x = gbl((const double*)(MODE == LP_ZERO ? L.r : (MODE == LP_STEP1 ? L.t : L.z)));
  auto* zout = gblw(MODE == LP_STEP0 || MODE == LP_RES ? L.t : L.z);
  auto* dd = gblw(L.d);
  // groups of cw lanes split the row's entries (V = 1; V = 4: one group)
  const int lane = (int)(threadIdx.x % LN);
  const int grp = V > 1 ? 0 : lane / cw, ngrp = V > 1 ? 1 : LN / cw;
  const int col0 = (V > 1 ? lane : lane - grp * cw) * V;
  const bool act = col0 < ncol;
  for (int64_t i = (int64_t)blockIdx.x * (NT / LN) + threadIdx.x / LN; i < L.N; i += (int64_t)gridDim.x * (NT / LN)) {
    double y[V], rv[V], xv[V], dv[V], di = 0.0;
#pragma unroll
    for (int v = 0; v < V; ++v) y[v] = 0.0;
    const int64_t e = i * ncol + col0;
    if (act) {
      load_vals<V>(r + e, rv);
      if constexpr (MODE == LP_STEP0 || MODE == LP_STEP1) load_vals<V>(x + e, xv);
      if constexpr (MODE == LP_STEP1) load_vals<V>((const __attribute__((address_space(1))) double*)dd + e, dv);
      if (MODE != LP_RES) di = dinv[i];
      const int beg = ptr[i] + grp, end = ptr[i + 1];
      if (end > beg) row_gather_v<V>(col, val, beg, end, ngrp, x, ncol, col0, y);
    }
    if constexpr (V == 1)
      for (int off = LN / 2; off >= cw; off >>= 1) y[0] += __shfl_xor(y[0], off, 64);
    if (!act || grp > 0) continue;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      if constexpr (MODE == LP_RES) {
        zout[e + v] = rv[v] - y[v];
      } else if constexpr (MODE == LP_ZERO) {
        const double z0 = c0 * di * rv[v];
        zout[e + v] = z0 + (c1 * z0 + c2 * di * (rv[v] - c0 * y[v]));
      } else if constexpr (MODE == LP_STEP0) {
        const double dn = c0 * di * (rv[v] - y[v]);
        dd[e + v] = dn;
        zout[e + v] = xv[v] + dn;
      } else {
        zout[e + v] = xv[v] + (c1 * dv[v] + c2 * di * (rv[v] - y[v]));
      }
    }
  }
}

template <int MODE>
static void coarse_pass(const MgDev& mg, int l, int ni, int ncol, hipStream_t s) {
  int cw = 1;
  while (cw < ncol) cw *= 2;
  auto go = [&](auto kern, int ln) {
    hipLaunchKernelGGL(kern, dim3(nblocks(mg.max_n[l] * ln, NT, 16384), ni), dim3(NT), 0, s, mg.lv[l], ncol, cw);
  };
  // Few columns: four lane groups share a row's entries where one lane per entry
  // and column leaves the chip idle (2^20 lanes: four waves' worth of every SIMD's
  // slots), since the longest rows, beside hanging nodes, then set the time.
  // Measured, one group -> four: 18,700 rows x 4 columns 10.1 -> 7.2 us a pass,
  // 16 x 34,000 rows x 4 columns 57 -> 72 us.
  const bool few = mg.max_n[l] * ni * cw < (int64_t)1 << 20;
  if (ncol >= 16 && ncol % 4 == 0) {
    if (ncol > 32) go(k_mg_level_pass<MODE, 4, 16>, 16);
    else if (ncol > 16) go(k_mg_level_pass<MODE, 4, 8>, 8);
    else go(k_mg_level_pass<MODE, 4, 4>, 4);
  } else if (cw == 1) few ? go(k_mg_level_pass<MODE, 1, 4>, 4) : go(k_mg_level_pass<MODE, 1, 1>, 1);
  else if (cw == 2) few ? go(k_mg_level_pass<MODE, 1, 8>, 8) : go(k_mg_level_pass<MODE, 1, 2>, 2);
  else if (cw == 4) few ? go(k_mg_level_pass<MODE, 1, 16>, 16) : go(k_mg_level_pass<MODE, 1, 4>, 4);
  else if (cw == 8) few ? go(k_mg_level_pass<MODE, 1, 32>, 32) : go(k_mg_level_pass<MODE, 1, 8>, 8);
  else if (cw == 16) few ? go(k_mg_level_pass<MODE, 1, 64>, 64) : go(k_mg_level_pass<MODE, 1, 16>, 16);
  else if (cw == 32) go(k_mg_level_pass<MODE, 1, 32>, 32);
  else go(k_mg_level_pass<MODE, 1, 64>, 64);
}

static void smooth(const MgDev& mg, int l, int ni, int ncol, bool from_zero, const MgLevel0Ops& ops, hipStream_t s) {
  if (l == 0) {  // fused into the level-0 operator passes (degree mg.nu >= 2)
    if (from_zero) {
      ops.cheb0(s);                                   // steps 0 and 1
      for (int k = 2; k < mg.nu; ++k) ops.cheb(k, false, s);
    } else {
      for (int k = 0; k < mg.nu; ++k) ops.cheb(k, k == mg.nu - 1, s);
    }
    return;
  }
  if (from_zero) {
    coarse_pass<LP_ZERO>(mg, l, ni, ncol, s);
  } else {
    coarse_pass<LP_STEP0>(mg, l, ni, ncol, s);
    coarse_pass<LP_STEP1>(mg, l, ni, ncol, s);
  }
}

// Hanging rows of a level's correction (z rows N .. N + Nh), so that the cells of
// the finer level read every coarse node's value directly.
__global__ void __launch_bounds__(NT) k_mg_fill(const MgLevelDev* __restrict__ lv, int ncol) {
  const MgLevelDev& L = lv[blockIdx.y];
  if (L.done && *L.done) return;
  const int64_t total = L.Nh * ncol;
  const auto* ptr = gbl(L.h_ptr);
  const auto* z = gbl((const double*)L.z);
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < total; e += (int64_t)gridDim.x * NT) {
    const int64_t h = e / ncol;
    const int c = (int)(e - h * ncol), beg = ptr[h], end = ptr[h + 1];
    gblw(L.z)[L.N * ncol + e] = end > beg ? row_gather_dot(gbl(L.h_col), gbl(L.h_w), beg, end, 1, z, ncol, c) : 0.0;
  }
}

// fine.z += P coarse.z where the two levels lie on the same leaves, PF and PC
// nodes per edge: a cell interpolates its PC^3 coarse nodes along z, y and x
// (B[a][b]: coarse basis function b at fine node a) and adds to the fine DoFs it
// is named for.  Row by row every fine node gathers up to PC^3 coarse rows, 12.7
// on average from Q2 to Q3; here a cell reads PC^3 rows for its share of the fine
// nodes (27 for 27).  Bound by the chain index -> row -> store, so a plane's rows
// are requested together; a thread takes a column of a cell, or (SPLIT) of one of
// its planes.  Rows -> cells, Q2 to
// Q3 and Q1 to Q2 together: H2O (1.5 M and 429,000 fine rows x 64 columns) 1333 ->
// 943 us (by planes 1066), 16 H2 (4 columns) 136 -> 68 us by planes (85 by cells).
struct InterpTable {
  double B[12];
};
template <int PF, int PC, bool SPLIT>
__global__ void __launch_bounds__(NT) k_mg_prolong_cells(const MgLevelDev* __restrict__ fine,
                                                         const MgLevelDev* __restrict__ coarse, int ncol,
                                                         InterpTable tab) {
  const MgLevelDev& F = fine[blockIdx.y];
  if (!F.active || (F.done && *F.done)) return;
  const auto* x = gbl((const double*)coarse[blockIdx.y].z);
  const auto* cf = gbl(F.cell_f);
  const auto* cc = gbl(F.cell_c);
  auto* z = gblw(F.z);
  auto* zf = gblw(F.zf);
  const bool f32 = F.f32 != 0;
  constexpr int PF3 = PF * PF * PF, PC3 = PC * PC * PC, NP = SPLIT ? PF : 1;
  const int total = (int)F.nC * NP, per = NT / ncol;   // ncol consecutive threads take a cell (plane)
  const int g = (int)threadIdx.x / ncol, c = (int)threadIdx.x - g * ncol;
  if (g >= per) return;
  const XcdSweep sw = xcd_sweep(total, per);
  for (int w = (int)sw.start + g; w < (int)sw.end; w += (int)sw.step) {
    const int64_t e = w / NP;
    const int plane = w - (int)e * NP;
    double u[PC3];
#pragma unroll
    for (int k = 0; k < PC3; ++k) {
      const int j = cc[e * PC3 + k];
      const double v = x[(int64_t)(j < 0 ? 0 : j) * ncol + c];
      u[k] = j < 0 ? 0.0 : v;
    }
#pragma unroll
    for (int q = 0; q < (SPLIT ? 1 : PF); ++q) {
      const int fz = SPLIT ? plane : q;
      int f[PF * PF];
#pragma unroll
      for (int k = 0; k < PF * PF; ++k) f[k] = cf[e * PF3 + fz * PF * PF + k];
      double zo[PF * PF], wz[PC * PC];
#pragma unroll
      for (int k = 0; k < PF * PF; ++k) {
        const int64_t o = (int64_t)(f[k] < 0 ? 0 : f[k]) * ncol + c;
        zo[k] = f32 ? (double)zf[o] : z[o];
      }
#pragma unroll
      for (int k = 0; k < PC * PC; ++k) {
        double t = 0.0;
#pragma unroll
        for (int m = 0; m < PC; ++m) t += tab.B[fz * PC + m] * u[m * PC * PC + k];
        wz[k] = t;
      }
#pragma unroll
      for (int fy = 0; fy < PF; ++fy) {
        double wy[PC];
#pragma unroll
        for (int k = 0; k < PC; ++k) {
          double t = 0.0;
#pragma unroll
          for (int m = 0; m < PC; ++m) t += tab.B[fy * PC + m] * wz[m * PC + k];
          wy[k] = t;
        }
#pragma unroll
        for (int fx = 0; fx < PF; ++fx) {
          double t = zo[fy * PF + fx];
#pragma unroll
          for (int m = 0; m < PC; ++m) t += tab.B[fx * PC + m] * wy[m];
          if (f[fy * PF + fx] >= 0) {
            const int64_t o = (int64_t)f[fy * PF + fx] * ncol + c;
            if (f32) zf[o] = (float)t;
            else z[o] = t;
          }
        }
      }
    }
  }
}

static void prolong_cells(const MgDev& mg, int l, int ni, int ncol, hipStream_t s) {
  const int pf = mg.cell_pf[l], pc = mg.cell_pc[l];
  if (mg.max_hang[l + 1] > 0)
    hipLaunchKernelGGL(k_mg_fill, dim3(nblocks(mg.max_hang[l + 1] * ncol, NT, 16384), ni), dim3(NT), 0, s, mg.lv[l + 1],
                       ncol);
  InterpTable tab{};
  for (int a = 0; a < pf; ++a)
    for (int b = 0; b < pc; ++b) tab.B[a * pc + b] = mg.interp[l][a * pc + b];
  // a thread per plane where the cells alone leave the chip idle (below 2^19 lanes;
  // between 2^17 and 2^20 it is much the same).  Cells, planes, Q2 to Q3: 11,300 lanes
  // (4 columns) 26.8, 10.6 us; 45,000 (16) 26.4, 12.9; 180,000 (64) 34.7, 39.6 and, 16
  // instances of 4 columns, 47.5, 50.8; 233,000 (4) 79.9, 63.5; 450,000 (40 instances)
  // 124, 116; 934,000 (16) 213, 224
  const bool split = mg.max_cells[l] * ncol * ni < (int64_t)1 << 19;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(xcd_grid(mg.max_cells[l] * (split ? pf : 1), NT / ncol, 65536), ni), dim3(NT), 0, s,
                       mg.lv[l], mg.lv[l + 1], ncol, tab);
  };
  if (pf == 4) split ? go(k_mg_prolong_cells<4, 3, true>) : go(k_mg_prolong_cells<4, 3, false>);
  else split ? go(k_mg_prolong_cells<3, 2, true>) : go(k_mg_prolong_cells<3, 2, false>);
}

void mg_vcycle(const MgDev& mg, int ni, int ncol, const MgLevel0Ops& ops, hipStream_t s) {
  const int nl = mg.nlev;
  // 4 columns per lane in the transfers when the column count is a multiple of
  // 4: for the restriction from 16 columns on (at 4 columns its 64 lane groups
  // spend more on combining than they gain), for the prolongation from 4 on
  const bool wide = ncol >= 16 && ncol % 4 == 0;
  const bool wide_p = ncol % 4 == 0;
  for (int l = 0; l + 1 < nl; ++l) {
    smooth(mg, l, ni, ncol, true, ops, s);
    // the residual r - A z that the restriction reads: the level-0 residual
    // pass, or the coarse level's fused pass
    if (l > 0) coarse_pass<LP_RES>(mg, l, ni, ncol, s);
    else ops.resid(s);
    if (wide) {
      int cw = 1;
      while (cw * 4 < ncol) cw *= 2;
      const dim3 g(xcd_grid(mg.max_n[l + 1], NT / 64, 16384), ni);
      hipLaunchKernelGGL(k_mg_restrict_v<4>, g, dim3(NT), 0, s, mg.lv[l], mg.lv[l + 1], ncol, cw);
    } else {
      int cw = 1;
      while (cw < ncol) cw *= 2;
      // lanes per row: four groups of them share its entries where the rows alone
      // fill the chip (at least 16 lanes), else the whole wave.  Whole wave, four
      // groups: 1,153 rows x 4 columns 4.9, 8.1 us; 1,979 4.6, 5.4; 7,916 8.8, 6.9;
      // 18,719 15.0, 13.7; 74,900 49.9, 33.4
      const int G = mg.max_n[l + 1] * ni >= 4096 ? std::min(64, std::max(16, 4 * cw)) : 64;
      hipLaunchKernelGGL(k_mg_restrict, dim3(xcd_grid(mg.max_n[l + 1], NT / G, 16384), ni), dim3(NT), 0, s, mg.lv[l],
                         mg.lv[l + 1], ncol, cw, G);
    }
  }
  {
    const dim3 g((unsigned)((mg.max_coarse + 15) / 16), ni);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, g, dim3(64 * MC_W), 0, s, mg.coarse, ncol); };
    if (ncol <= 16) go(k_mg_coarse<1>);
    else if (ncol <= 32) go(k_mg_coarse<2>);
    else if (ncol <= 48) go(k_mg_coarse<3>);
    else go(k_mg_coarse<4>);
  }
  for (int l = nl - 2; l >= 0; --l) {
    if (mg.cell_pf[l])
      prolong_cells(mg, l, ni, ncol, s);
    else if (wide_p && ncol > 32)
      hipLaunchKernelGGL((k_mg_prolong_v<4, 16>), dim3(xcd_grid(mg.max_n[l], NT / 16, 16384), ni), dim3(NT), 0, s,
                         mg.lv[l], mg.lv[l + 1], ncol);
    else if (wide_p && ncol > 16)
      hipLaunchKernelGGL((k_mg_prolong_v<4, 8>), dim3(xcd_grid(mg.max_n[l], NT / 8, 16384), ni), dim3(NT), 0, s,
                         mg.lv[l], mg.lv[l + 1], ncol);
    else if (wide_p && ncol > 4)
      hipLaunchKernelGGL((k_mg_prolong_v<4, 4>), dim3(xcd_grid(mg.max_n[l], NT / 4, 16384), ni), dim3(NT), 0, s,
                         mg.lv[l], mg.lv[l + 1], ncol);
    else if (wide_p)
      hipLaunchKernelGGL((k_mg_prolong_v<4, 1>), dim3(xcd_grid(mg.max_n[l], NT, 16384), ni), dim3(NT), 0, s,
                         mg.lv[l], mg.lv[l + 1], ncol);
    else
      hipLaunchKernelGGL(k_mg_prolong, level_grid(mg.max_n[l], ncol, ni), dim3(NT), 0, s, mg.lv[l], mg.lv[l + 1],
                         ncol);
    smooth(mg, l, ni, ncol, false, ops, s);
  }
}

// red[i][slot] = r . z per instance and column (overwrites)
__global__ void __launch_bounds__(NT) k_rz_parts(const DevMesh* __restrict__ dm, int ncol, const double* __restrict__ r,
                                                 const double* __restrict__ z, double* __restrict__ part) {
  INSTANCE;
  // ncol consecutive threads take one row (coalesced), NT / ncol rows per pass
  __shared__ double lds[NT];
  r += d.oE * ncol;
  z += d.oE * ncol;
  const int groups = NT / ncol;
  const int g = threadIdx.x / ncol, c = threadIdx.x - g * ncol;
  double acc = 0.0;
  if (g < groups)
    for (int64_t i = (int64_t)blockIdx.x * groups + g; i < d.N; i += (int64_t)gridDim.x * groups)
      acc += r[i * ncol + c] * z[i * ncol + c];
  lds[threadIdx.x] = g < groups ? acc : 0.0;
  __syncthreads();
  if (threadIdx.x < (unsigned)ncol) {
    double t = 0.0;
    for (int q = 0; q < groups; ++q) t += lds[q * ncol + threadIdx.x];
    part[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * ncol + threadIdx.x] = t;
  }
}
__global__ void __launch_bounds__(NT) k_rz_finish(const double* __restrict__ part, int nblk, int ncol,
                                                  double* __restrict__ red, int slot) {
  __shared__ double lds4[4];
  const int c = blockIdx.x;
  part += (int64_t)blockIdx.y * nblk * ncol;
  red += (int64_t)blockIdx.y * RED_SLOTS * ncol;
  const double v = sum_partials(part, nblk, ncol, c, lds4);
  if (threadIdx.x == 0) red[slot * ncol + c] = v;
}
void mg_rz(const DevMesh* dm, int ni, int ncol, const double* r, const double* z, double* part, double* red, int slot,
           hipStream_t s) {
  hipLaunchKernelGGL(k_rz_parts, dim3(MG_RZ_BLOCKS, ni), dim3(NT), 0, s, dm, ncol, r, z, part);
  hipLaunchKernelGGL(k_rz_finish, dim3(ncol, ni), dim3(NT), 0, s, part, MG_RZ_BLOCKS, ncol, red, slot);
}

// The deferred solution update of the last CG iteration: x += alpha p with
// alpha from the r.z slot rz_slot and the p.q slot pq_slot.
__global__ void __launch_bounds__(NT) k_cg_xfinal(const DevMesh* __restrict__ dm, int ncol, double* __restrict__ x,
                                                  const double* __restrict__ p, const double* __restrict__ red,
                                                  int rz_slot, int pq_slot) {
  INSTANCE;
  __shared__ double alpha[64];
  red += (int64_t)blockIdx.y * RED_SLOTS * ncol;
  if (threadIdx.x < (unsigned)ncol) {
    const double rz = red[rz_slot * ncol + threadIdx.x], pq = red[pq_slot * ncol + threadIdx.x];
    alpha[threadIdx.x] = (pq != 0.0 && rz != 0.0) ? rz / pq : 0.0;
  }
  __syncthreads();
  x += d.oF * ncol;
  p += d.oE * ncol;
  const int64_t total = d.N * ncol;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < total; e += (int64_t)gridDim.x * NT)
    x[e] += alpha[e % ncol] * p[e];
}
void cg_xfinal(const DevMesh* dm, int ni, int64_t max_n, int ncol, double* x, const double* p, const double* red,
               int rz_slot, int pq_slot, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_xfinal, dim3(nblocks(max_n * ncol, NT, 8192), ni), dim3(NT), 0, s, dm, ncol, x, p, red,
                     rz_slot, pq_slot);
}

}  // namespace mh
