// HIP kernels of the MCTDHF-on-octree-FEM hot path for gfx950 (wave64):
// interface mass solve, constraint fill, reductions, mean-field build,
// Krylov (Arnoldi) pieces, Poisson right-hand side and multipole boundary
// values, small dense work and the CI space.
//
// Orbital arrays are complex128 [rows][n] (orbital fastest); Poisson arrays
// are real [rows][ncol].  Row space of one instance: [0,N) DoFs, [N,NE)
// hanging nodes, [NE,NF) box-boundary nodes.  Batched launches: instance
// blockIdx.y, batch row offsets from its DevMesh (kernels.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "devutil.hpp"
#include "kernels.hpp"

namespace mh {

// Sum over a 256-thread block; result valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double* lds) {
  v = wave_sum(v);
  int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) lds[wid] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0) t = lds[0] + lds[1] + lds[2] + lds[3];
  return t;
}

#define INSTANCE const DevMesh& d = dm[blockIdx.y]

// =====================================================================
// Chebyshev iteration on the interface block A_Ma (Jacobi-preconditioned,
// spectrum bounds from set-up): x_{k+1} = x_k + d_k, r_{k+1} = r_k - A d_k,
// d_{k+1} = c1_k d_k + c2_k D^-1 r_{k+1}; the per-instance coefficients
// (from that instance's bounds) are tabulated in d.cheb.
// =====================================================================
__global__ void __launch_bounds__(NT) k_cheb_init(const DevMesh* __restrict__ dm, const double2* __restrict__ b,
                                                  double2* __restrict__ x, double2* __restrict__ r,
                                                  double2* __restrict__ d0) {
  INSTANCE;
  const int n = d.n;
  const int64_t total = d.nMa * n, o = d.oMa * n;
  if (total == 0) return;
  const double inv_theta = d.cheb[0];
  for (int64_t idx = (int64_t)blockIdx.x * NT + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * NT) {
    const int64_t i = idx / n;
    double2 bi = b[o + idx];
    x[o + idx] = make_double2(0.0, 0.0);
    r[o + idx] = bi;
    d0[o + idx] = cscale(d.ma_dinv[i] * inv_theta, bi);
  }
}

// One Chebyshev step on the interface block, a row per four groups of NP lanes (25
// entries a row at Q3, 9 at Q1).  Bound by the chain row -> index -> gather: the
// matrix and the vectors (10 and 21 MB at H2O) stay in the caches.  Eight lanes
// a row, each gathering whole orbital rows (one 16-byte load per lane and
// orbital, scattered) -> an orbital per lane, a launch: H2O (33,344 rows x 8
// orbitals) 31.6 -> 17.8 us, its Q1 mesh (12,746 x 8) 10.5 -> 6.2 us, 16 H2
// (2,382 x 2 each) 11.7 -> 11.0 us (thirty-two lanes a row: 19.0, 7.5, 14.1 us).
template <int NP>
__global__ void __launch_bounds__(NT) k_cheb_iter(const DevMesh* __restrict__ dm, double2* __restrict__ x,
                                                  double2* __restrict__ r, const double2* __restrict__ din,
                                                  double2* __restrict__ dout, int k) {
  INSTANCE;
  constexpr int LR = 4 * NP;
  const int n = d.n;
  if (d.nMa == 0) return;
  const int64_t o = d.oMa * n;
  const double c1 = d.cheb[1 + 2 * k], c2 = d.cheb[2 + 2 * k];
  const int lane = (int)(threadIdx.x & (LR - 1));
  const auto* mp = gbl(d.ma_ptr);
  // XCD x sweeps the x-th eighth of the (band-ordered) rows, so its gathers
  // stay within that part of the vectors and hit its own L2
  const XcdSweep sw = xcd_sweep(d.nMa, NT / LR);
  for (int64_t i = sw.start + threadIdx.x / LR; i < sw.end; i += sw.step) {
    const int beg = mp[i], end = mp[i + 1];
    double2 dk = make_double2(0.0, 0.0), xi = dk, ri = dk;
    double gi = 0.0;
    const int64_t idx = o + i * n + lane;
    if (lane < n) {
      dk = ldg2(din, idx);
      xi = ldg2((const double2*)x, idx);
      ri = ldg2((const double2*)r, idx);
      gi = c2 * gbl(d.ma_dinv)[i];
    }
    const double2 q = orb_row<NP, LR, 4>(d.ma_col, d.ma_val, beg, end, INT32_MAX, din + o, n);
    if (lane < n) {
      const double2 rn = csub(ri, q);
      x[idx] = cadd(xi, dk);
      r[idx] = rn;
      dout[idx] = make_double2(c1 * dk.x + gi * rn.x, c1 * dk.y + gi * rn.y);
    }
  }
}

__global__ void __launch_bounds__(NT) k_cheb_finish(const DevMesh* __restrict__ dm, const double2* __restrict__ x,
                                                    const double2* __restrict__ dk, const double2* __restrict__ v,
                                                    const double2* __restrict__ lam, double2* __restrict__ out) {
  INSTANCE;
  const int n = d.n;
  const int64_t total = d.nMa * n, o = d.oMa * n, oe = d.oE * n;
  const double2* L = lam ? lam + (int64_t)blockIdx.y * n * n : nullptr;
  for (int64_t idx = (int64_t)blockIdx.x * NT + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * NT) {
    const int64_t i = idx / n;
    const int p = (int)(idx - i * n);
    const int64_t k = d.ma_dof[i];
    double2 xf = cadd(x[o + idx], dk[o + idx]);
    if (L)
      for (int q = 0; q < n; ++q) xf = csub(xf, cmul(L[q * n + p], v[oe + k * n + q]));
    out[oe + k * n + p] = xf;
  }
}

// Interface solve by the dense inverse (one instance): x = A^-1 b, R rows per
// workgroup, its four waves splitting the columns; then the final value of each
// master DoF as in k_cheb_finish.  NP: the orbital count rounded up (2, 4 or 8).
// Bound by the inverse (45 MB at H2's 2,382 masters).  A wave per row read b once
// a row, four times the inverse's bytes, with nine waves a CU; here b is read
// once for R rows: H2 (2,382 masters x 2 orbitals) 16.5 -> 11.9 us, three orbitals
// on a Q2 mesh 12.2 -> 8.6 us.
// LOAD: the solve of a given load vector (b over extended rows): the right-hand
// side is read through the masters' DoFs, and the workgroups from `dense` on
// divide the other DoFs by their mass, which saves the gathering launch.
template <int NP, int R, bool LOAD>
__global__ void __launch_bounds__(NT) k_ma_dense(const DevMesh* __restrict__ dm, const double2* __restrict__ b,
                                                 const double2* __restrict__ v, const double2* __restrict__ lam,
                                                 double2* __restrict__ out, int dense) {
  INSTANCE;
  if (LOAD && (int)blockIdx.x >= dense) {
    const int64_t total = d.N * d.n, od = d.oE * d.n;
    for (int64_t e = (int64_t)((int)blockIdx.x - dense) * NT + threadIdx.x; e < total;
         e += (int64_t)((int)gridDim.x - dense) * NT) {
      const int64_t k = e / d.n;
      const double2 f = ldg2(b, od + e);
      const double im = gbl(d.inv_mass)[k];
      if (gbl(d.ma_index)[k] < 0) out[od + e] = cscale(im, f);
    }
    return;
  }
  constexpr int W = NT / 64;
  __shared__ double part[W][R * NP * 2];
  const int n = d.n, nMa = (int)d.nMa;
  const int64_t o = d.oMa * n, oe = d.oE * n;
  const auto* Ai = gbl(d.ma_inv);
  const double2* L = lam ? lam + (int64_t)blockIdx.y * n * n : nullptr;
  for (int i0 = (int)blockIdx.x * R; i0 < nMa; i0 += dense * R) {
    double s[R * NP * 2];
#pragma unroll
    for (int k = 0; k < R * NP * 2; ++k) s[k] = 0.0;
    int64_t row[R];
#pragma unroll
    for (int r = 0; r < R; ++r) row[r] = (int64_t)min(i0 + r, nMa - 1) * nMa;
    // two strides of the workgroup's columns in flight; columns past the end
    // repeat the last one with coefficient zero
    for (int j0 = (int)threadIdx.x; j0 < nMa; j0 += 2 * NT) {
      double a[2][R];
      double2 bj[2][NP];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int j = j0 + u * NT, jc = min(j, nMa - 1);
#pragma unroll
        for (int r = 0; r < R; ++r) a[u][r] = Ai[row[r] + jc];
#pragma unroll
        for (int p = 0; p < NP; ++p)
          bj[u][p] = ldg2(b, (LOAD ? oe + (int64_t)gbl(d.ma_dof)[jc] * n : o + (int64_t)jc * n) + min(p, n - 1));
        if (j >= nMa) {
#pragma unroll
          for (int r = 0; r < R; ++r) a[u][r] = 0.0;
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            s[(r * NP + p) * 2] += a[u][r] * bj[u][p].x;
            s[(r * NP + p) * 2 + 1] += a[u][r] * bj[u][p].y;
          }
    }
    wave_sum_values(s, part[threadIdx.x >> 6]);
    __syncthreads();
    const int r = (int)threadIdx.x / NP, p = (int)threadIdx.x - r * NP, i = i0 + r;
    if (r < R && p < n && i < nMa) {
      double2 xf = make_double2(0.0, 0.0);
#pragma unroll
      for (int w = 0; w < W; ++w) {
        xf.x += part[w][(r * NP + p) * 2];
        xf.y += part[w][(r * NP + p) * 2 + 1];
      }
      const int64_t k = d.ma_dof[i];
      if (L)
        for (int q = 0; q < n; ++q) xf = csub(xf, cmul(L[q * n + p], v[oe + k * n + q]));
      out[oe + k * n + p] = xf;
    }
    __syncthreads();
  }
}

// In-place inverse of a dense SPD matrix by Gauss-Jordan steps of GJ_B pivots at
// once, K the block of rows and columns k0 .. k0 + GJ_B: A_KK <- A_KK^-1 ...
constexpr int GJ_B = 32, GJ_T = 64;
__global__ void __launch_bounds__(NT) k_gj_pivot(double* __restrict__ A, int64_t n, int64_t k0) {
  __shared__ double row[2][GJ_B], col[2][GJ_B];
  const int b = (int)min((int64_t)GJ_B, n - k0), j = (int)threadIdx.x % GJ_B, i0 = (int)threadIdx.x / GJ_B;
  constexpr int M = GJ_B * GJ_B / NT, S = NT / GJ_B;   // rows i0, i0 + S, ... of column j
  double a[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int i = i0 + S * m;
    a[m] = i < b && j < b ? A[(k0 + i) * n + k0 + j] : (i == j ? 1.0 : 0.0);   // past the end: the identity
  }
  for (int p = 0; p < b; ++p) {
    double *r = row[p & 1], *c = col[p & 1];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int i = i0 + S * m;
      if (i == p) r[j] = a[m];
      if (j == p) c[i] = a[m];
    }
    __syncthreads();
    const double inv = 1.0 / r[p], rj = r[j];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int i = i0 + S * m;
      const double ci = c[i];
      a[m] = i == p ? (j == p ? inv : rj * inv) : (j == p ? -ci * inv : a[m] - ci * rj * inv);
    }
  }
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int i = i0 + S * m;
    if (i < b && j < b) A[(k0 + i) * n + k0 + j] = a[m];
  }
}
// ... then (COL = false) A_Kj <- A_KK^-1 A_Kj for the columns j outside K, or (COL =
// true, after the update below) A_iK <- -A_iK A_KK^-1 for the rows i outside K:
// GJ_T columns (rows) a workgroup, a thread one of them and GJ_B / 4 sums ...
template <bool COL>
__global__ void __launch_bounds__(NT) k_gj_panel(double* __restrict__ A, int64_t n, int64_t k0) {
  __shared__ double P[GJ_B][GJ_B + 1], X[GJ_T][GJ_B + 1];
  const int b = (int)min((int64_t)GJ_B, n - k0);
  const int64_t t0 = (int64_t)blockIdx.x * GJ_T;
  for (int e = threadIdx.x; e < GJ_B * GJ_B; e += NT) {
    const int i = e / GJ_B, j = e % GJ_B;
    P[i][j] = i < b && j < b ? A[(k0 + i) * n + k0 + j] : 0.0;
  }
  for (int e = threadIdx.x; e < GJ_T * GJ_B; e += NT) {
    const int t = COL ? e / GJ_B : e % GJ_T, k = COL ? e % GJ_B : e / GJ_T;
    const bool ok = t0 + t < n && k < b;
    X[t][k] = ok ? A[COL ? (t0 + t) * n + k0 + k : (k0 + k) * n + t0 + t] : 0.0;
  }
  __syncthreads();
  const int t = (int)threadIdx.x % GJ_T, g = (int)threadIdx.x / GJ_T;
  constexpr int M = GJ_B / (NT / GJ_T);
  double y[M];
#pragma unroll
  for (int m = 0; m < M; ++m) y[m] = 0.0;
  for (int k = 0; k < GJ_B; ++k) {
    const double x = X[t][k];
#pragma unroll
    for (int m = 0; m < M; ++m) y[m] += (COL ? -P[k][g * M + m] : P[g * M + m][k]) * x;
  }
  const int64_t at = t0 + t;
  if (at >= n || (at >= k0 && at < k0 + b)) return;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int k = g * M + m;
    if (k < b) A[COL ? at * n + k0 + k : (k0 + k) * n + at] = y[m];
  }
}
// ... and A_ij <- A_ij - A_iK A_Kj (the new A_Kj) for i and j outside K, GJ_T x GJ_T
// entries a workgroup, 4 x 4 a thread.  Bound by the launches (four per block of
// pivots) and the pivot block's chain.  A pivot at a time took three launches each,
// all n^2 entries read and written in every first one: 2,382 unknowns 57 -> 6.4 ms,
// 1,979 36.5 -> 4.6 ms, 1,153 12.5 -> 2.3 ms (launching them took up to twice that).
// Against the inverse in extended precision, of condition 1.5 and 1,000: 1.0e-15 and
// 2.9e-14 a pivot at a time, 0.3e-15 and 1.2e-14 by blocks (500 unknowns)
__global__ void __launch_bounds__(NT) k_gj_update(double* __restrict__ A, int64_t n, int64_t k0) {
  __shared__ double C[GJ_B][GJ_T + 1], R[GJ_B][GJ_T + 1];
  const int b = (int)min((int64_t)GJ_B, n - k0);
  const int64_t i0 = (int64_t)blockIdx.y * GJ_T, j0 = (int64_t)blockIdx.x * GJ_T;
  for (int e = threadIdx.x; e < GJ_T * GJ_B; e += NT) {
    const int ti = e / GJ_B, k = e % GJ_B, tj = e % GJ_T, l = e / GJ_T;
    C[k][ti] = i0 + ti < n && k < b ? A[(i0 + ti) * n + k0 + k] : 0.0;
    R[l][tj] = j0 + tj < n && l < b ? A[(k0 + l) * n + j0 + tj] : 0.0;
  }
  __syncthreads();
  const int tx = (int)threadIdx.x % 16, ty = (int)threadIdx.x / 16;
  double y[4][4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) y[u][v] = 0.0;
#pragma unroll 8
  for (int k = 0; k < GJ_B; ++k) {
    double c[4], r[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      c[u] = C[k][ty + 16 * u];
      r[u] = R[k][tx + 16 * u];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) y[u][v] += c[u] * r[v];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t i = i0 + ty + 16 * u;
    if (i >= n || (i >= k0 && i < k0 + b)) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t j = j0 + tx + 16 * v;
      if (j < n && !(j >= k0 && j < k0 + b)) A[i * n + j] -= y[u][v];
    }
  }
}
void launch_dense_inverse(double* A, int64_t n, hipStream_t s) {
  const unsigned t = (unsigned)((n + GJ_T - 1) / GJ_T);
  for (int64_t k0 = 0; k0 < n; k0 += GJ_B) {
    hipLaunchKernelGGL(k_gj_pivot, dim3(1), dim3(NT), 0, s, A, n, k0);
    if (n <= GJ_B) break;
    hipLaunchKernelGGL(k_gj_panel<false>, dim3(t), dim3(NT), 0, s, A, n, k0);
    hipLaunchKernelGGL(k_gj_update, dim3(t, t), dim3(NT), 0, s, A, n, k0);
    hipLaunchKernelGGL(k_gj_panel<true>, dim3(t), dim3(NT), 0, s, A, n, k0);
  }
}

void launch_ma_solve(const Batch& b, const double* ma_b, double* x, double* r, double* dbuf0, double* dbuf1,
                     const double* v, const double* lam, double* out, hipStream_t s) {
  if (b.mx.nMa == 0) return;
  if (b.ni == 1 && b.mx.ma_inv && !(b.mx.sched_orb & 2)) {
    auto go = [&](auto kern, int rows) {
      const int g = nblocks(b.mx.nMa, rows, 8192);
      hipLaunchKernelGGL(kern, dim3(g), dim3(NT), 0, s, b.dm, (const double2*)ma_b, (const double2*)v,
                         (const double2*)lam, (double2*)out, g);
    };
    if (b.mx.n <= 2) go(k_ma_dense<2, 4, false>, 4);
    else if (b.mx.n <= 4) go(k_ma_dense<4, 4, false>, 4);
    else go(k_ma_dense<8, 2, false>, 2);
    return;
  }
  const dim3 g(nblocks(b.mx.nMa * b.mx.n), b.ni);
  hipLaunchKernelGGL(k_cheb_init, g, dim3(NT), 0, s, b.dm, (const double2*)ma_b, (double2*)x, (double2*)r,
                     (double2*)dbuf0);
  double* din = dbuf0;
  double* dout = dbuf1;
  for (int k = 0; k < b.cheb_iters; ++k) {
    orb_dispatch(b.mx.n, [&](auto np) {
      const dim3 gi(xcd_grid(b.mx.nMa, NT / (4 * np.value), 65536), b.ni);
      hipLaunchKernelGGL(k_cheb_iter<np.value>, gi, dim3(NT), 0, s, b.dm, (double2*)x, (double2*)r,
                         (const double2*)din, (double2*)dout, k);
    });
    double* t = din;
    din = dout;
    dout = t;
  }
  hipLaunchKernelGGL(k_cheb_finish, g, dim3(NT), 0, s, b.dm, (const double2*)x, (const double2*)din,
                     (const double2*)v, (const double2*)lam, (double2*)out);
}

// Mass solve of a load vector f (extended rows) on the DoFs: with a dense inverse
// one launch, the non-masters' workgroups beside the dense rows'; in place, and on
// the Chebyshev path, the masters' rows are gathered to ma_b first.  H atom (4,007
// DoFs, 196 masters), hanging rows included: three launches -> two, 9.5 -> 6.8 us on
// the device, 14.0 -> 11.0 us a call.  Each workgroup then gathers the masters' rows of
// f through their DoFs, so with many of them the launch that lays them out first
// is the cheaper: masters x orbitals of 670 x 8 12.4 us against 15.0 laid out, 1,220 x 4
// 11.4 against 13.3, 2,382 x 2 18.7 against 18.2, 1,220 x 5 19.5 against 15.0, 2,382 x 3
// 23.2 against 21.0, x 5 53.1 against 39.7.
constexpr int64_t MA_LOAD_MAX = 5400;
void launch_mass_solve(const Batch& b, const double* f, double* out, double* ma_b, double* x, double* r, double* dbuf0,
                       double* dbuf1, hipStream_t s) {
  if (b.ni == 1 && b.mx.nMa > 0 && b.mx.ma_inv && !(b.mx.sched_orb & 2) && f != out &&
      b.mx.nMa * b.mx.n <= MA_LOAD_MAX) {
    auto go = [&](auto kern, int rows) {
      const int g = nblocks(b.mx.nMa, rows, 8192);
      hipLaunchKernelGGL(kern, dim3(g + nblocks(b.mx.N * b.mx.n, NT, 8192)), dim3(NT), 0, s, b.dm, (const double2*)f,
                         (const double2*)nullptr, (const double2*)nullptr, (double2*)out, g);
    };
    if (b.mx.n <= 2) go(k_ma_dense<2, 4, true>, 4);
    else if (b.mx.n <= 4) go(k_ma_dense<4, 4, true>, 4);
    else go(k_ma_dense<8, 2, true>, 2);
    return;
  }
  launch_mass_direct(b, f, out, ma_b, s);
  launch_ma_solve(b, ma_b, x, r, dbuf0, dbuf1, nullptr, nullptr, out, s);
}

// Hanging rows: x[h] = sum_k c_hk x[k] over DoF masters (boundary values of
// orbitals vanish); optionally zero the hanging rows of acc.  A row per
// four groups of NP lanes: the masters (12.6 on average at Q3) are gathered in one round
// instead of one after the other by a thread per orbital: H2 (9,240 rows x 2
// orbitals) 9.8 -> 4.7 us, 16 of it 26.8 -> 13.8 us, H2O (129,640 x 8) 31.7 -> 32.4 us.
template <int NP>
__global__ void __launch_bounds__(NT) k_fill_orb(const DevMesh* __restrict__ dm, double2* __restrict__ x,
                                                 double2* __restrict__ acc) {
  INSTANCE;
  constexpr int LR = 4 * NP;
  const int n = d.n;
  const int64_t o = d.oE * n;
  const int lane = (int)(threadIdx.x & (LR - 1));
  const auto* hp = gbl(d.hang_ptr);
  const XcdSweep sw = xcd_sweep(d.Nh, NT / LR);
  for (int64_t h = sw.start + threadIdx.x / LR; h < sw.end; h += sw.step) {
    const double2 s = orb_row<NP, LR, 4>(d.hang_col, d.hang_w, hp[h], hp[h + 1], (int)d.N, x + o, n);
    if (lane < n) {
      x[o + (d.N + h) * n + lane] = s;
      if (acc) acc[o + (d.N + h) * n + lane] = make_double2(0.0, 0.0);
    }
  }
}

void launch_fill_orb(const Batch& b, double* x, double* acc, hipStream_t s) {
  if (b.mx.Nh == 0) return;
  orb_dispatch(b.mx.n, [&](auto np) {
    hipLaunchKernelGGL(k_fill_orb<np.value>, dim3(xcd_grid(b.mx.Nh, NT / (4 * np.value), 65536), b.ni), dim3(NT), 0, s, b.dm,
                       (double2*)x, (double2*)acc);
  });
}

__global__ void k_copy(const double* __restrict__ in, double* __restrict__ out, int64_t nd) {
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < nd; i += (int64_t)gridDim.x * NT) out[i] = in[i];
}
__global__ void k_zero(double* __restrict__ out, int64_t nd) {
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < nd; i += (int64_t)gridDim.x * NT) out[i] = 0.0;
}
__global__ void k_set(double* __restrict__ out, double value) {
  if (threadIdx.x == 0 && blockIdx.x == 0) out[0] = value;
}
void launch_copy(const double* in, double* out, int64_t nd, hipStream_t s) {
  if (nd > 0) hipLaunchKernelGGL(k_copy, dim3(nblocks(nd, NT, 8192)), dim3(NT), 0, s, in, out, nd);
}
void launch_zero(double* out, int64_t nd, hipStream_t s) {
  if (nd > 0) hipLaunchKernelGGL(k_zero, dim3(nblocks(nd, NT, 8192)), dim3(NT), 0, s, out, nd);
}
// x <- 2 x - xp and xp <- the old x (linear extrapolation in time, history shifted)
__global__ void k_extrapolate(double* __restrict__ x, double* __restrict__ xp, int64_t nd) {
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < nd; i += (int64_t)gridDim.x * NT) {
    const double xi = x[i];
    x[i] = 2.0 * xi - xp[i];
    xp[i] = xi;
  }
}
void launch_extrapolate(double* x, double* xprev, int64_t nd, hipStream_t s) {
  if (nd > 0) hipLaunchKernelGGL(k_extrapolate, dim3(nblocks(nd, NT, 8192)), dim3(NT), 0, s, x, xprev, nd);
}
// x <- 3 x - 3 p1 + p2 (quadratic extrapolation in time), then p2 <- p1, p1 <- the old x
__global__ void k_extrapolate2(double* __restrict__ x, double* __restrict__ p1, double* __restrict__ p2, int64_t nd) {
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < nd; i += (int64_t)gridDim.x * NT) {
    const double xi = x[i], a = p1[i];
    x[i] = 3.0 * (xi - a) + p2[i];
    p2[i] = a;
    p1[i] = xi;
  }
}
void launch_extrapolate2(double* x, double* p1, double* p2, int64_t nd, hipStream_t s) {
  if (nd > 0) hipLaunchKernelGGL(k_extrapolate2, dim3(nblocks(nd, NT, 8192)), dim3(NT), 0, s, x, p1, p2, nd);
}
void launch_set(double* out, double value, hipStream_t s) {
  hipLaunchKernelGGL(k_set, dim3(1), dim3(64), 0, s, out, value);
}
// A step counter on the device, so that a captured step reads its own field
// value from a table: out = table[*ctr]; ctr += add.
__global__ void k_set_indexed(double* __restrict__ out, const double* __restrict__ table,
                              const int* __restrict__ ctr) {
  if (threadIdx.x == 0 && blockIdx.x == 0) out[0] = table[ctr[0]];
}
__global__ void k_counter(int* __restrict__ ctr, int set, int value) {
  if (threadIdx.x == 0 && blockIdx.x == 0) ctr[0] = set ? value : ctr[0] + value;
}
void launch_set_indexed(double* out, const double* table, const int* ctr, hipStream_t s) {
  hipLaunchKernelGGL(k_set_indexed, dim3(1), dim3(64), 0, s, out, table, ctr);
}
void launch_counter(int* ctr, int set, int value, hipStream_t s) {
  hipLaunchKernelGGL(k_counter, dim3(1), dim3(64), 0, s, ctr, set, value);
}

// =====================================================================
// Tiled reduction: out[a][b] = sum_i wt_i conj(X[i][a]) Y[i][b], one output set
// per instance.  X, Y are batch orbital arrays with na, nb columns, rows N or NE
// of the instance, weight none / m / m z.  Partials per block, then a finishing pass.  Deterministic.
// =====================================================================
constexpr int XG_CH = 16;
__global__ void __launch_bounds__(NT) k_xgram(const DevMesh* __restrict__ dm, int wsel, int rsel,
                                              const double2* __restrict__ X, int na, const double2* __restrict__ Y,
                                              int nb, double2* __restrict__ part) {
  __shared__ double2 sx[XG_CH * 64];
  __shared__ double2 sy[XG_CH * 64];
  INSTANCE;
  const int64_t rows = rsel == ROWS_EXT ? d.NE : d.N;
  const double* wt = wsel == WT_MASS ? d.m : (wsel == WT_DIPOLE ? d.mz : nullptr);
  X += d.oE * na;
  Y += d.oE * nb;
  const int nout = na * nb;
  constexpr int MAXO = 16;  // outputs per thread (na*nb <= 4096)
  double2 accv[MAXO];
#pragma unroll
  for (int j = 0; j < MAXO; ++j) accv[j] = make_double2(0.0, 0.0);
  for (int64_t base = (int64_t)blockIdx.x * XG_CH; base < rows; base += (int64_t)gridDim.x * XG_CH) {
    const int cnt = (int)((rows - base) < XG_CH ? (rows - base) : XG_CH);
    __syncthreads();
    for (int e = threadIdx.x; e < XG_CH * na; e += NT) {
      int r = e / na, a = e - r * na;
      double2 v = make_double2(0.0, 0.0);
      if (r < cnt) {
        v = X[(base + r) * na + a];
        if (wt) v = cscale(gbl(wt)[base + r], v);
      }
      sx[r * na + a] = v;
    }
    for (int e = threadIdx.x; e < XG_CH * nb; e += NT) {
      int r = e / nb, bb = e - r * nb;
      sy[r * nb + bb] = (r < cnt) ? Y[(base + r) * nb + bb] : make_double2(0.0, 0.0);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < MAXO; ++j) {
      int o = threadIdx.x + j * NT;
      if (o >= nout) break;
      int a = o / nb, bb = o - a * nb;
      double2 s = accv[j];
      for (int r = 0; r < cnt; ++r) {
        double2 xv = sx[r * na + a], yv = sy[r * nb + bb];
        s.x += xv.x * yv.x + xv.y * yv.y;
        s.y += xv.x * yv.y - xv.y * yv.x;
      }
      accv[j] = s;
    }
  }
  double2* pb = part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * nout;
#pragma unroll
  for (int j = 0; j < MAXO; ++j) {
    int o = threadIdx.x + j * NT;
    if (o < nout) pb[o] = accv[j];
  }
}

// The same for small output sets (na nb <= 16): every thread accumulates all
// outputs over a grid-stride set of rows (no staging, no barrier per chunk),
// then one reduction per workgroup (shuffles, then the four waves).
__global__ void __launch_bounds__(NT) k_xgram_small(const DevMesh* __restrict__ dm, int wsel, int rsel,
                                                    const double2* __restrict__ X, int na,
                                                    const double2* __restrict__ Y, int nb,
                                                    double2* __restrict__ part) {
  __shared__ double2 lw[NT / 64][16];
  INSTANCE;
  const int64_t rows = rsel == ROWS_EXT ? d.NE : d.N;
  const double* wt = wsel == WT_MASS ? d.m : (wsel == WT_DIPOLE ? d.mz : nullptr);
  X += d.oE * na;
  Y += d.oE * nb;
  const int nout = na * nb;
  double2 acc[16];
#pragma unroll
  for (int o = 0; o < 16; ++o) acc[o] = make_double2(0.0, 0.0);
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < rows; i += (int64_t)gridDim.x * NT) {
    const double w = wt ? gbl(wt)[i] : 1.0;
#pragma unroll
    for (int o = 0; o < 16; ++o)
      if (o < nout) {
        const int a = o / nb, bb = o - a * nb;
        const double2 xv = cscale(w, X[i * na + a]), yv = Y[i * nb + bb];
        acc[o].x += xv.x * yv.x + xv.y * yv.y;
        acc[o].y += xv.x * yv.y - xv.y * yv.x;
      }
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int o = 0; o < 16; ++o)
    if (o < nout) {
      const double sx = wave_sum(acc[o].x), sy = wave_sum(acc[o].y);
      if (lane == 0) lw[wid][o] = make_double2(sx, sy);
    }
  __syncthreads();
  if (threadIdx.x < (unsigned)nout) {
    double2 t = lw[0][threadIdx.x];
    for (int w = 1; w < NT / 64; ++w) t = cadd(t, lw[w][threadIdx.x]);
    part[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * nout + threadIdx.x] = t;
  }
}

// out[o] = sum over nblk partials [nblk][nout] (per instance): cw consecutive
// outputs per workgroup, its NT / cw slices of the partials summed in turn (eight
// loads in flight) and folded in LDS, so that a partial's outputs are read in
// whole lines.  Bound by HBM on long partials, by the launch on short ones.  A
// workgroup per output reading with the partials' stride -> this, at 8 orbitals:
// moments (2,048 partials of 10,816) 234 us, pair integrals (8,192 outputs) and Gram
// matrices (128) 55 us on average -> all 14 launches of two steps 1130 -> 145 us; 8
// outputs 3.1 -> 3.0 us.
__global__ void __launch_bounds__(NT) k_sum_parts(const double* __restrict__ part, int nblk, int nout, int cw,
                                                  double* __restrict__ out) {
  __shared__ double lds[NT];
  const int c = (int)threadIdx.x % cw, g = (int)threadIdx.x / cw, G = NT / cw;
  const int o = (int)blockIdx.x * cw + c, oc = min(o, nout - 1);
  const auto* p = gbl(part + (int64_t)blockIdx.y * nblk * nout);
  double s = 0.0;
  for (int b = g; b < nblk; b += 8 * G) {
    double v[8];
#pragma unroll
    for (int h = 0; h < 8; ++h) v[h] = p[(int64_t)min(b + h * G, nblk - 1) * nout + oc];
#pragma unroll
    for (int h = 0; h < 8; ++h) s += b + h * G < nblk ? v[h] : 0.0;
  }
  lds[threadIdx.x] = s;
  __syncthreads();
  for (int h = G / 2; h > 0; h >>= 1) {
    if (g < h) lds[threadIdx.x] += lds[threadIdx.x + h * cw];
    __syncthreads();
  }
  if (g == 0 && o < nout) out[(int64_t)blockIdx.y * nout + o] = lds[c];
}
// 16 outputs (a 128-byte line) a workgroup where that still gives a workgroup
// per quarter of the chip, else 4: then a thread has one round of loads.
static void launch_sum_parts(const double* part, int nblk, int nout, double* out, int ni, hipStream_t s) {
  const int cw = nout >= 1024 ? 16 : 4;
  hipLaunchKernelGGL(k_sum_parts, dim3((nout + cw - 1) / cw, ni), dim3(NT), 0, s, part, nblk, nout, cw, out);
}

int gram_blocks(int64_t rows) { return nblocks(rows, XG_CH, 512); }

void launch_gram(const Batch& b, const double* A, const double* B, int wsel, int rows, double* part, int nblk,
                 double* G, hipStream_t s) {
  const int n = b.mx.n;
  if (n * n <= 16)
    hipLaunchKernelGGL(k_xgram_small, dim3(nblk, b.ni), dim3(NT), 0, s, b.dm, wsel, rows, (const double2*)A, n,
                       (const double2*)B, n, (double2*)part);
  else
    hipLaunchKernelGGL(k_xgram, dim3(nblk, b.ni), dim3(NT), 0, s, b.dm, wsel, rows, (const double2*)A, n,
                       (const double2*)B, n, (double2*)part);
  launch_sum_parts(part, nblk, 2 * n * n, G, b.ni, s);
}

// Pair-product integrals: G[(p,q)][col] = sum_i m_i conj(phi_p) phi_q Wcol_i
// (X built on the fly as phi_p conj(phi_q) so that conj(X) = conj(phi_p) phi_q).
// Register tiles of GT_A pair products x GT_C columns per thread: every
// round of LDS reads (four products, four potentials) feeds 32 FMAs; tiles
// numbered column-tile fastest, at most NT of them (n <= 8).
constexpr int GT_A = 4, GT_C = 4;
__global__ void __launch_bounds__(NT) k_gint(const DevMesh* __restrict__ dm, const double2* __restrict__ phi,
                                             const double* __restrict__ W, int ncol, double2* __restrict__ part) {
  INSTANCE;
  __shared__ double2 sx[XG_CH * 64];
  __shared__ double sw[XG_CH * 64];
  const int n = d.n, na = n * n, nout = na * ncol;
  const int nap = (na + GT_A - 1) / GT_A * GT_A, ncp = (ncol + GT_C - 1) / GT_C * GT_C;
  phi += d.oE * n;
  W += d.oF * ncol;
  const int tiles_c = ncp / GT_C, tiles = (nap / GT_A) * tiles_c;
  const bool act = (int)threadIdx.x < tiles;
  const int a0 = act ? ((int)threadIdx.x / tiles_c) * GT_A : 0, c0 = act ? ((int)threadIdx.x % tiles_c) * GT_C : 0;
  double2 acc[GT_A][GT_C];
#pragma unroll
  for (int u = 0; u < GT_A; ++u)
#pragma unroll
    for (int v = 0; v < GT_C; ++v) acc[u][v] = make_double2(0.0, 0.0);
  const int64_t rows = d.NE;
  for (int64_t base = (int64_t)blockIdx.x * XG_CH; base < rows; base += (int64_t)gridDim.x * XG_CH) {
    const int cnt = (int)((rows - base) < XG_CH ? (rows - base) : XG_CH);
    __syncthreads();
    for (int e = threadIdx.x; e < XG_CH * nap; e += NT) {
      const int r = e / nap, a = e - r * nap;
      double2 v = make_double2(0.0, 0.0);
      if (r < cnt && a < na) {
        const int p = a / n, q = a - p * n;
        const int64_t i = base + r;
        const double2 fp = phi[i * n + p], fq = phi[i * n + q];
        // phi_p conj(phi_q) * m_i
        v = cscale(d.m[i], make_double2(fp.x * fq.x + fp.y * fq.y, fp.y * fq.x - fp.x * fq.y));
      }
      sx[r * nap + a] = v;
    }
    for (int e = threadIdx.x; e < XG_CH * ncp; e += NT) {
      const int r = e / ncp, c = e - r * ncp;
      sw[r * ncp + c] = (r < cnt && c < ncol) ? W[(base + r) * ncol + c] : 0.0;
    }
    __syncthreads();
    if (act)
      for (int r = 0; r < cnt; ++r) {
        double2 xv[GT_A];
        double yv[GT_C];
#pragma unroll
        for (int u = 0; u < GT_A; ++u) xv[u] = sx[r * nap + a0 + u];
#pragma unroll
        for (int v = 0; v < GT_C; ++v) yv[v] = sw[r * ncp + c0 + v];
#pragma unroll
        for (int u = 0; u < GT_A; ++u)
#pragma unroll
          for (int v = 0; v < GT_C; ++v) {
            acc[u][v].x += xv[u].x * yv[v];
            acc[u][v].y -= xv[u].y * yv[v];
          }
      }
  }
  if (!act) return;
  double2* pb = part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * nout;
#pragma unroll
  for (int u = 0; u < GT_A; ++u)
#pragma unroll
    for (int v = 0; v < GT_C; ++v)
      if (a0 + u < na && c0 + v < ncol) pb[(a0 + u) * ncol + c0 + v] = acc[u][v];
}

// The same on the matrix cores (n >= 4): per chunk of GM_CH rows the real
// and imaginary parts of the products X and the potentials are staged in
// LDS, and Re G = sum Re X W, Im G = -sum Im X W accumulate in FP64 MFMA tiles
// of 16 products x 16 columns (the lane layout of k_moments_mfma), the tiles
// (real and imaginary product tiles x column tiles) dealt round-robin to the
// four waves, at most GM_TW per wave.
constexpr int GM_CH = 16, GM_TW = 8;
typedef double dvec4g_t __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(NT) k_gint_mfma(const DevMesh* __restrict__ dm, const double2* __restrict__ phi,
                                                  const double* __restrict__ W, int ncol,
                                                  double2* __restrict__ part) {
  INSTANCE;
  __shared__ double sxr[GM_CH * 64];
  __shared__ double sxi[GM_CH * 64];
  __shared__ double sw[GM_CH * 64];
  const int n = d.n, na = n * n, nout = na * ncol;
  phi += d.oE * n;
  W += d.oF * ncol;
  const int nat = (na + 15) / 16, nct = (ncol + 15) / 16, ntile = 2 * nat * nct;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  dvec4g_t acc[GM_TW];
#pragma unroll
  for (int j = 0; j < GM_TW; ++j) acc[j] = dvec4g_t{0.0, 0.0, 0.0, 0.0};
  const int64_t rows = d.NE;
  for (int64_t base = (int64_t)blockIdx.x * GM_CH; base < rows; base += (int64_t)gridDim.x * GM_CH) {
    const int cnt = (int)((rows - base) < GM_CH ? (rows - base) : GM_CH);
    __syncthreads();
    for (int e = threadIdx.x; e < GM_CH * 64; e += NT) {
      const int r = e >> 6, a = e & 63;
      double xr = 0.0, xi = 0.0, wv = 0.0;
      if (r < cnt) {
        const int64_t i = base + r;
        if (a < na) {
          const int p = a / n, q = a - p * n;
          const double2 fp = phi[i * n + p], fq = phi[i * n + q];
          const double mi = d.m[i];
          // m_i phi_p conj(phi_q)
          xr = mi * (fp.x * fq.x + fp.y * fq.y);
          xi = mi * (fp.y * fq.x - fp.x * fq.y);
        }
        if (a < ncol) wv = W[i * ncol + a];
      }
      sxr[e] = xr;
      sxi[e] = xi;
      sw[e] = wv;
    }
    __syncthreads();
#pragma unroll
    for (int k0 = 0; k0 < GM_CH; k0 += 4) {
      const int kr = k0 + (lane >> 4), li = lane & 15;
#pragma unroll
      for (int j = 0; j < GM_TW; ++j) {
        const int tile = wave + 4 * j;
        if (tile < ntile) {
          const int u = tile % nct, ta = tile / nct;   // ta < nat: real tiles, then imaginary
          const int t = ta < nat ? ta : ta - nat;
          const double a = (ta < nat ? sxr : sxi)[kr * 64 + 16 * t + li];
          const double b = sw[kr * 64 + 16 * u + li];
          acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[j], 0, 0, 0);
        }
      }
    }
  }
  double* pb = (double*)(part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * nout);
#pragma unroll
  for (int j = 0; j < GM_TW; ++j) {
    const int tile = wave + 4 * j;
    if (tile >= ntile) continue;
    const int u = tile % nct, ta = tile / nct;
    const bool im = ta >= nat;
    const int t = im ? ta - nat : ta;
    const int c = 16 * u + (lane & 15);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = 16 * t + 4 * v + (lane >> 4);
      // conj(X) W: the imaginary part enters with a minus sign
      if (a < na && c < ncol) pb[2 * (a * ncol + c) + (im ? 1 : 0)] = im ? -acc[j][v] : acc[j][v];
    }
  }
}

// The same for n^2 x ncol <= 16 outputs (two orbitals): every thread
// accumulates all outputs over a grid-stride set of rows, then one reduction
// per workgroup.
__global__ void __launch_bounds__(NT) k_gint_small(const DevMesh* __restrict__ dm, const double2* __restrict__ phi,
                                                   const double* __restrict__ W, int ncol,
                                                   double2* __restrict__ part) {
  INSTANCE;
  __shared__ double2 lw[NT / 64][16];
  const int n = d.n, na = n * n, nout = na * ncol;
  phi += d.oE * n;
  W += d.oF * ncol;
  double2 acc[16];
#pragma unroll
  for (int o = 0; o < 16; ++o) acc[o] = make_double2(0.0, 0.0);
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < d.NE; i += (int64_t)gridDim.x * NT) {
    const double mi = gbl(d.m)[i];
#pragma unroll
    for (int o = 0; o < 16; ++o)
      if (o < nout) {
        const int a = o / ncol, c = o - a * ncol;
        const int p = a / n, q = a - p * n;
        const double2 fp = phi[i * n + p], fq = phi[i * n + q];
        // phi_p conj(phi_q) m_i, conjugated
        const double2 xv = cscale(mi, make_double2(fp.x * fq.x + fp.y * fq.y, fp.y * fq.x - fp.x * fq.y));
        const double yv = W[i * ncol + c];
        acc[o].x += xv.x * yv;
        acc[o].y -= xv.y * yv;
      }
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int o = 0; o < 16; ++o)
    if (o < nout) {
      const double sx = wave_sum(acc[o].x), sy = wave_sum(acc[o].y);
      if (lane == 0) lw[wid][o] = make_double2(sx, sy);
    }
  __syncthreads();
  if (threadIdx.x < (unsigned)nout) {
    double2 t = lw[0][threadIdx.x];
    for (int w = 1; w < NT / 64; ++w) t = cadd(t, lw[w][threadIdx.x]);
    part[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * nout + threadIdx.x] = t;
  }
}

// Assemble g_pqrs from the pair-column integrals G[(p,q)][col].
__global__ void k_gint_assemble(const double2* __restrict__ G, int n, const int* __restrict__ colmap,
                                double2* __restrict__ g) {
  const int ncol = n * n, n4 = ncol * ncol;
  G += (int64_t)blockIdx.y * n4;
  g += (int64_t)blockIdx.y * n4;
  for (int o = blockIdx.x * NT + threadIdx.x; o < n4; o += gridDim.x * NT) {
    int s = o % n, r = (o / n) % n, pq = o / (n * n);
    int rr = r < s ? r : s, ss = r < s ? s : r;
    int cre = colmap[rr * n + ss];
    double2 val = G[pq * ncol + cre];
    if (rr != ss) {
      double2 im = G[pq * ncol + cre + 1];
      double sg = (r < s) ? 1.0 : -1.0;
      val = make_double2(val.x - sg * im.y, val.y + sg * im.x);
    }
    g[o] = val;
  }
}

// up to 2048 workgroups for the matrix-core form (n >= 4), 512 otherwise
int gint_blocks(const Batch& b) { return nblocks(b.mx.NE, XG_CH, b.mx.n >= 4 ? 2048 : 512); }

void launch_gint_full(const Batch& b, const double* phi, const double* W, const int* colmap, double* part, int nblk,
                      double* Gtmp, double* g, hipStream_t s) {
  const int n = b.mx.n, ncol = n * n;
  if (ncol * ncol <= 16)
    hipLaunchKernelGGL(k_gint_small, dim3(nblk, b.ni), dim3(NT), 0, s, b.dm, (const double2*)phi, W, ncol,
                       (double2*)part);
  else if (n >= 4)   // matrix cores: at least one full 16 x 16 tile
    hipLaunchKernelGGL(k_gint_mfma, dim3(nblk, b.ni), dim3(NT), 0, s, b.dm, (const double2*)phi, W, ncol,
                       (double2*)part);
  else
    hipLaunchKernelGGL(k_gint, dim3(nblk, b.ni), dim3(NT), 0, s, b.dm, (const double2*)phi, W, ncol,
                       (double2*)part);
  launch_sum_parts(part, nblk, 2 * ncol * ncol, Gtmp, b.ni, s);
  hipLaunchKernelGGL(k_gint_assemble, dim3(nblocks(ncol * ncol), b.ni), dim3(NT), 0, s, (const double2*)Gtmp, n,
                     colmap, (double2*)g);
}

// =====================================================================
// Mean field: U(x) = sum_rs Gamma_oq,rs W_rs(x), a real linear map of the
// n^2 real Poisson columns to the n^2 packed entries of the Hermitian U.
// =====================================================================
__global__ void k_build_Mreal(const double2* __restrict__ Gamma, int n, const int* __restrict__ colmap,
                              double* __restrict__ Mr) {
  const int nn = n * n;
  Gamma += (int64_t)blockIdx.y * nn * nn;
  Mr += (int64_t)blockIdx.y * nn * nn;
  for (int o = blockIdx.x * NT + threadIdx.x; o < nn * nn; o += gridDim.x * NT) {
    int out = o / nn, col = o - out * nn;
    int oi = out / n, qi = out - oi * n;  // packed position
    int ro = oi < qi ? oi : qi, co = oi < qi ? qi : oi;
    bool want_im = oi > qi;               // lower triangle holds the imaginary part
    // locate (r, s, part) of col
    int rr = 0, ss = 0, part = 0;
    for (int r = 0; r < n; ++r)
      for (int s = r; s < n; ++s) {
        int c0 = colmap[r * n + s];
        if (c0 == col) { rr = r; ss = s; part = 0; }
        if (r != s && c0 + 1 == col) { rr = r; ss = s; part = 1; }
      }
    // U_{ro,co} as a function of column value: Gamma_{ro co, rr ss} (a + i b) + Gamma_{ro co, ss rr} (a - i b)
    double2 g1 = Gamma[((ro * n + co) * n + rr) * n + ss];
    double2 g2 = Gamma[((ro * n + co) * n + ss) * n + rr];
    double2 coef;
    if (rr == ss) coef = g1;                                      // a only
    else if (part == 0) coef = cadd(g1, g2);                       // d U / d a
    else coef = make_double2(-(g1.y - g2.y), g1.x - g2.x);          // i (g1 - g2)
    Mr[o] = want_im ? coef.y : coef.x;
  }
}

// Upk[i][o] = sum_c Mr[o][c] W[i][c]: G lanes per node (G = n^2 rounded up
// to a power of two), lane o owning output o; the node's W row is read once,
// coalesced, and broadcast by shuffles; Mr is held transposed in LDS so the
// lanes of a group read consecutive words.
template <int G>
__global__ void __launch_bounds__(NT) k_build_U(const DevMesh* __restrict__ dm, const double* __restrict__ W,
                                                const double* __restrict__ Mr, double* __restrict__ Upk) {
  INSTANCE;
  __shared__ double sMT[64 * 64];
  const int nn = d.n * d.n;
  Mr += (int64_t)blockIdx.y * nn * nn;
  W += d.oF * nn;
  Upk += d.oE * nn;
  for (int e = threadIdx.x; e < nn * nn; e += NT) {
    const int o = e / nn, c = e - o * nn;
    sMT[c * nn + o] = Mr[e];
  }
  __syncthreads();
  const int o = (int)(threadIdx.x & (G - 1));
  for (int64_t i = ((int64_t)blockIdx.x * NT + threadIdx.x) / G; i < d.NE; i += ((int64_t)gridDim.x * NT) / G) {
    const double w = o < nn ? W[i * nn + o] : 0.0;
    double acc = 0.0;
    for (int c = 0; c < nn; ++c) {
      const double wc = __shfl(w, c, G);
      if (o < nn) acc += sMT[c * nn + o] * wc;
    }
    if (o < nn) Upk[i * nn + o] = acc;
  }
}

// Eight orbitals (64 x 64 map) on the matrix cores: per chunk of 64 rows, wave w takes rows
// 16 w .. 16 w + 15 and all four 16-output tiles, U = W M^T accumulated in
// FP64 MFMA tiles (lane layout of k_moments_mfma) over the 64 columns, four
// per instruction; W rows staged in LDS (row stride 65), M transposed in LDS.
typedef double dvec4u_t __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(NT) k_build_U64_mfma(const DevMesh* __restrict__ dm, const double* __restrict__ W,
                                                       const double* __restrict__ Mr, double* __restrict__ Upk) {
  INSTANCE;
  __shared__ double sMT[64 * 64];
  __shared__ double sW[64 * 65];
  Mr += (int64_t)blockIdx.y * 64 * 64;
  W += d.oF * 64;
  Upk += d.oE * 64;
  for (int e = threadIdx.x; e < 64 * 64; e += NT) {
    const int o = e >> 6, c = e & 63;
    sMT[c * 64 + o] = Mr[e];
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  for (int64_t base = (int64_t)blockIdx.x * 64; base < d.NE; base += (int64_t)gridDim.x * 64) {
    const int cnt = (int)((d.NE - base) < 64 ? (d.NE - base) : 64);
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * 64; e += NT) {
      const int r = e >> 6, c = e & 63;
      sW[r * 65 + c] = r < cnt ? W[(base + r) * 64 + c] : 0.0;
    }
    __syncthreads();
    dvec4u_t acc[4];
#pragma unroll
    for (int ot = 0; ot < 4; ++ot) acc[ot] = dvec4u_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int c0 = 0; c0 < 64; c0 += 4) {
      const double a = sW[(16 * wave + li) * 65 + c0 + lk];
#pragma unroll
      for (int ot = 0; ot < 4; ++ot) {
        const double bv = sMT[(c0 + lk) * 64 + 16 * ot + li];
        acc[ot] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bv, acc[ot], 0, 0, 0);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * wave + 4 * v + lk;
      if (r < cnt)
#pragma unroll
        for (int ot = 0; ot < 4; ++ot) Upk[(base + r) * 64 + 16 * ot + li] = acc[ot][v];
    }
  }
}

void launch_build_U_full(const Batch& b, const double* W, const double* Gamma, const int* colmap, double* Mr,
                         double* Upk, hipStream_t s) {
  const int nn = b.mx.n * b.mx.n;
  hipLaunchKernelGGL(k_build_Mreal, dim3(nblocks(nn * nn), b.ni), dim3(NT), 0, s, (const double2*)Gamma, b.mx.n,
                     colmap, Mr);
  const int g = nblocks(b.mx.NE * 64, NT, 8192);
  if (nn <= 1) hipLaunchKernelGGL(k_build_U<1>, dim3(g, b.ni), dim3(NT), 0, s, b.dm, W, Mr, Upk);
  else if (nn <= 4) hipLaunchKernelGGL(k_build_U<4>, dim3(g, b.ni), dim3(NT), 0, s, b.dm, W, Mr, Upk);
  else if (nn <= 16) hipLaunchKernelGGL(k_build_U<16>, dim3(g, b.ni), dim3(NT), 0, s, b.dm, W, Mr, Upk);
  else if (nn < 64) hipLaunchKernelGGL(k_build_U<64>, dim3(g, b.ni), dim3(NT), 0, s, b.dm, W, Mr, Upk);
  else hipLaunchKernelGGL(k_build_U64_mfma, dim3(nblocks(b.mx.NE, 64, 8192), b.ni), dim3(NT), 0, s, b.dm, W, Mr, Upk);
}

// =====================================================================
// Krylov (Arnoldi) pieces.  M-inner product over the packed orbital vector:
// <u,v> = sum_i m_i sum_p conj(u_ip) v_ip on rows [0, NE) of each instance.
// Per-instance strides: H (m_max+1) m_max, y m_max, scal 8,
// partials nblk (2 (m_max+1) + 1).
// =====================================================================
constexpr int KMAX = 25;

__device__ __forceinline__ int64_t kpart_stride(int nblk, int m_max) { return (int64_t)nblk * (2 * (m_max + 1) + 1); }

// Row of element e of a packed array of n (1..8) values per row: division by a
// constant in each branch (n is uniform), which a multiplication replaces.
__device__ __forceinline__ int64_t row_of(int64_t e, int n) {
  switch (n) {
    case 1: return e;
    case 2: return e >> 1;
    case 3: return (int64_t)((uint64_t)e / 3u);
    case 4: return e >> 2;
    case 5: return (int64_t)((uint64_t)e / 5u);
    case 6: return (int64_t)((uint64_t)e / 6u);
    case 7: return (int64_t)((uint64_t)e / 7u);
    default: return e >> 3;
  }
}

// A new basis vector takes three launches: the dots of the first Gram-Schmidt
// pass (k_mdot), the update with the decision on a second pass (k_orth) and
// the second update, where one is taken, with the normalisation (k_orth_scale).
// Each launch leaves one partial sum per workgroup and value, [value][workgroup],
// and the next one folds them: every workgroup for itself on short vectors
// (Krylov::fold, at most 256 partials per value, so the fold reads tens of KB
// from L2 and saves a launch), else a launch of its own with one workgroup per
// value (k_kry_fold), since hundreds of MB would be read again on long vectors.
// Measured against eight launches per vector (a fold, the decision, the norm
// and the scaling apart): H2 (151,750 elements)
// Arnoldi step 1296 -> 1156 us, H2O (13.2 M elements) 18.1 -> 14.0 ms in these
// passes over two steps
constexpr int KT = 512;   // threads of these passes
constexpr int KNV = 2 * KMAX + 1;

// Sum over the workgroup of one value, returned to every thread.
__device__ __forceinline__ double kry_sum(double v, double* lds) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < KT / 64; ++w) t += lds[w];
  return t;
}

template <int KM>
__global__ void __launch_bounds__(KT) k_mdot(const DevMesh* __restrict__ dm, const double2* const* __restrict__ V,
                                             int k, const double2* __restrict__ w, int m_max,
                                             double* __restrict__ part) {
  INSTANCE;
  constexpr int NV = 2 * KM + 1;
  __shared__ double lw[KT / 64][NV];
  const int n = d.n;
  const int64_t total = d.NE * n, o = d.oE * n;
  double acc[NV];   // Re, Im of the dot with each V_j, then |w|^2 last
#pragma unroll
  for (int j = 0; j < NV; ++j) acc[j] = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * KT + threadIdx.x; e < total; e += (int64_t)gridDim.x * KT) {
    const double mi = gbl(d.m)[row_of(e, n)];
    const double2 w0 = ldg2(w, o + e);
    const double2 we = make_double2(mi * w0.x, mi * w0.y);
#pragma unroll
    for (int j = 0; j < KM; ++j) {
      if (j <= k) {
        const double2 vj = ldg2(V[j], o + e);
        acc[2 * j] += vj.x * we.x + vj.y * we.y;
        acc[2 * j + 1] += vj.x * we.y - vj.y * we.x;
      }
    }
    acc[NV - 1] += we.x * w0.x + we.y * w0.y;
  }
  wave_sum_values(acc, lw[threadIdx.x >> 6]);
  __syncthreads();
  const int nv = 2 * (k + 1) + 1;
  if (threadIdx.x < (unsigned)nv) {
    const int v = (int)threadIdx.x < nv - 1 ? (int)threadIdx.x : NV - 1;
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < KT / 64; ++w) t += lw[w][v];
    part[blockIdx.y * kpart_stride(gridDim.x, m_max) + (int64_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
  }
}

// sums[v] = sum over the workgroups b of part[v][b], v < nv, by one workgroup
// (16 lanes per value, eight loads in flight), valid to every thread on return.
__device__ __forceinline__ void fold_values(const double* __restrict__ part, int nblk, int nv, double* sums) {
  const int g = threadIdx.x >> 4, l = threadIdx.x & 15;
  const auto* pg = gbl(part);
  for (int v = g; v < nv; v += KT / 16) {
    double s = 0.0;
    for (int b = l; b < nblk; b += 128) {
      double t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int bb = b + 16 * u;
        const double x = pg[(int64_t)v * nblk + (bb < nblk ? bb : b)];
        t[u] = bb < nblk ? x : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) s += t[u];
    }
    s += row_rotate<8>(s);
    s += row_rotate<4>(s);
    s += row_rotate<2>(s);
    s += row_rotate<1>(s);
    if (l == 0) sums[v] = s;
  }
  __syncthreads();
}

// The same as a launch: sums[i][v] of instance i, one workgroup per value.
// second: the sums of the second pass, which only instances that take one need.
__global__ void __launch_bounds__(NT) k_kry_fold(const double* __restrict__ part, int nblk, int m_max,
                                                 double* __restrict__ sums, const double* __restrict__ scal,
                                                 int second) {
  __shared__ double lds4[4];
  const int i = blockIdx.y, v = blockIdx.x;
  if (second && scal[8 * i + 6] != 0.0) return;
  const double s = sum_partials(part + i * kpart_stride(nblk, m_max) + (int64_t)v * nblk, nblk, 1, 0, lds4);
  if (threadIdx.x == 0) sums[(int64_t)i * (2 * (m_max + 1) + 1) + v] = s;
}

// First Gram-Schmidt update w -= sum_j V_j h_j from the dots of k_mdot, then
// the partials of |w|^2 and, where a second pass is taken, of V^H M w.
// Whether the first pass suffices is the criterion of Daniel, Gragg, Kaufman
// and Stewart 1976 on the norm the pass keeps: with the basis orthonormal,
// |w - V h|^2 = |w|^2 - sum |h_j|^2.  One pass leaves the new vector
// orthogonal to the basis to about the dots' rounding error times
// |w| / |w - V h| (measured on random bases of 200,000 rows: 6e-16 at a kept
// fraction of 0.7, 5e-15 at 0.1), so while the pass keeps at least a tenth of
// |w| (1/100 of |w|^2) the second pass is skipped (scal[6] = 1).
// KM >= k + 1 sizes the register arrays.
template <int KM>
__global__ void __launch_bounds__(KT) k_orth(const DevMesh* __restrict__ dm, const double2* const* __restrict__ V,
                                             int k, double2* __restrict__ w, int m_max, int fold,
                                             const double* __restrict__ part1, const double* __restrict__ sums1,
                                             double* __restrict__ part2, double2* __restrict__ H,
                                             double* __restrict__ scal) {
  INSTANCE;
  constexpr int NV = 2 * KM + 1;
  __shared__ double lw[KT / 64][NV];
  __shared__ double hs[KNV];
  const int n = d.n, inst = blockIdx.y;
  const int64_t total = d.NE * n, o = d.oE * n;
  const int nv = 2 * (k + 1) + 1;
  part2 += inst * kpart_stride(gridDim.x, m_max);
  if (fold) {
    fold_values(part1 + inst * kpart_stride(gridDim.x, m_max), gridDim.x, nv, hs);
  } else {
    if (threadIdx.x < (unsigned)nv) hs[threadIdx.x] = sums1[(int64_t)inst * (2 * (m_max + 1) + 1) + threadIdx.x];
    __syncthreads();
  }
  double2 h[KM];
  double hsq = 0.0;
#pragma unroll
  for (int j = 0; j < KM; ++j) {
    h[j] = make_double2(0.0, 0.0);
    if (j <= k) h[j] = make_double2(uniform(hs[2 * j]), uniform(hs[2 * j + 1]));
    hsq += h[j].x * h[j].x + h[j].y * h[j].y;
  }
  const double w2 = uniform(hs[nv - 1]);
  const bool single = w2 > 0.0 && w2 - hsq >= 0.01 * w2;
  if (blockIdx.x == 0 && threadIdx.x < (unsigned)nv) {
    double* Hk = (double*)(H + (int64_t)inst * (m_max + 1) * m_max + (int64_t)(m_max + 1) * k);
    if (threadIdx.x < (unsigned)(nv - 1)) {
      Hk[threadIdx.x] = hs[threadIdx.x];
    } else {
      scal[8 * inst + 2] = w2;
      scal[8 * inst + 6] = single ? 1.0 : 0.0;
    }
  }
  if (single) {
    double nrm = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * KT + threadIdx.x; e < total; e += (int64_t)gridDim.x * KT) {
      double2 we = ldg2(w, o + e);
#pragma unroll
      for (int j = 0; j < KM; ++j)
        if (j <= k) we = csub(we, cmul(h[j], ldg2(V[j], o + e)));
      w[o + e] = we;
      nrm += gbl(d.m)[row_of(e, n)] * (we.x * we.x + we.y * we.y);
    }
    const double c = kry_sum(nrm, &lw[0][0]);
    if (threadIdx.x == 0) part2[(int64_t)(nv - 1) * gridDim.x + blockIdx.x] = c;
    return;
  }
  double acc[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) acc[j] = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * KT + threadIdx.x; e < total; e += (int64_t)gridDim.x * KT) {
    double2 we = ldg2(w, o + e);
#pragma unroll
    for (int j = 0; j < KM; ++j)
      if (j <= k) we = csub(we, cmul(h[j], ldg2(V[j], o + e)));
    w[o + e] = we;
    const double mi = gbl(d.m)[row_of(e, n)];
    const double2 wm = make_double2(mi * we.x, mi * we.y);
    // the basis values are read again (from cache): kept, their registers would
    // halve the waves of the usual branch above
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < KM; ++j)
      if (j <= k) {
        const double2 vj = ldg2(V[j], o + e);
        acc[2 * j] += vj.x * wm.x + vj.y * wm.y;
        acc[2 * j + 1] += vj.x * wm.y - vj.y * wm.x;
      }
    acc[NV - 1] += wm.x * we.x + wm.y * we.y;
  }
  wave_sum_values(acc, lw[threadIdx.x >> 6]);
  __syncthreads();
  if (threadIdx.x < (unsigned)nv) {
    const int v = (int)threadIdx.x < nv - 1 ? (int)threadIdx.x : NV - 1;
    double t = 0.0;
#pragma unroll
    for (int w8 = 0; w8 < KT / 64; ++w8) t += lw[w8][v];
    part2[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
  }
}

// The new basis vector: the second update where one is taken, scaled by
// 1 / h_{k+1,k}, h_{k+1,k} = |w|; happy breakdown when h <= 1e-14 |G v_k| (then
// scale 0).  After a second pass |w|^2 is the first pass's norm less the
// squares of the second dots, which are rounding-sized against it (the two
// are comparable only where w itself is rounding noise, the breakdown).
// nblk: partials per value of k_orth.
template <int KM>
__global__ void __launch_bounds__(KT) k_orth_scale(const DevMesh* __restrict__ dm,
                                                   const double2* const* __restrict__ V, int k,
                                                   double2* __restrict__ w, int m_max, int fold, int nblk,
                                                   const double* __restrict__ part2,
                                                   const double* __restrict__ sums2, double2* __restrict__ H,
                                                   double* __restrict__ scal) {
  INSTANCE;
  __shared__ double lds[KT / 64];
  __shared__ double hs[KNV];
  const int n = d.n, inst = blockIdx.y;
  const int64_t total = d.NE * n, o = d.oE * n;
  const int nv = 2 * (k + 1) + 1;
  part2 += inst * kpart_stride(nblk, m_max);
  H += (int64_t)inst * (m_max + 1) * m_max + (int64_t)(m_max + 1) * k;
  scal += 8 * inst;
  const bool single = scal[6] != 0.0;
  double nrm2 = 0.0;
  if (single) {
    for (int b = threadIdx.x; b < nblk; b += KT) nrm2 += part2[(int64_t)(nv - 1) * nblk + b];
    nrm2 = kry_sum(nrm2, lds);
  } else {
    if (fold) {
      fold_values(part2, nblk, nv, hs);
    } else {
      if (threadIdx.x < (unsigned)nv) hs[threadIdx.x] = sums2[(int64_t)inst * (2 * (m_max + 1) + 1) + threadIdx.x];
      __syncthreads();
    }
    nrm2 = hs[nv - 1];
    for (int v = 0; v < nv - 1; ++v) nrm2 -= hs[v] * hs[v];
  }
  const double hn = nrm2 > 0.0 ? sqrt(nrm2) : (nrm2 == nrm2 ? 0.0 : nrm2);   // NaN stays NaN
  const bool brk = hn <= 1e-14 * sqrt(scal[2]) || !(hn > 0.0);
  const double sc = brk ? 0.0 : 1.0 / hn;
  if (blockIdx.x == 0) {
    if (!single && threadIdx.x < (unsigned)(nv - 1)) ((double*)H)[threadIdx.x] += hs[threadIdx.x];
    if (threadIdx.x == 0) {
      H[k + 1] = make_double2(hn, 0.0);
      if (brk && scal[4] > k + 1) scal[4] = k + 1;
    }
  }
  if (single) {
    for (int64_t e = (int64_t)blockIdx.x * KT + threadIdx.x; e < total; e += (int64_t)gridDim.x * KT)
      w[o + e] = cscale(sc, ldg2(w, o + e));
    return;
  }
  double2 h[KM];
#pragma unroll
  for (int j = 0; j < KM; ++j) {
    h[j] = make_double2(0.0, 0.0);
    if (j <= k) h[j] = make_double2(uniform(hs[2 * j]), uniform(hs[2 * j + 1]));
  }
  for (int64_t e = (int64_t)blockIdx.x * KT + threadIdx.x; e < total; e += (int64_t)gridDim.x * KT) {
    double2 we = ldg2(w, o + e);
#pragma unroll
    for (int j = 0; j < KM; ++j)
      if (j <= k) we = csub(we, cmul(h[j], ldg2(V[j], o + e)));
    w[o + e] = cscale(sc, we);
  }
}

template <int KM>
static void orthogonalize(const Batch& b, double* const* V, int k, double* w, Krylov& K, hipStream_t s) {
  const dim3 g(K.nblk, b.ni);
  const auto* Vc = (const double2* const*)V;
  const int nv = 2 * (k + 1) + 1, fold = K.fold ? 1 : 0;
  hipLaunchKernelGGL(k_mdot<KM>, g, dim3(KT), 0, s, b.dm, Vc, k, (const double2*)w, K.m_max, K.part);
  if (!fold)
    hipLaunchKernelGGL(k_kry_fold, dim3(nv, b.ni), dim3(NT), 0, s, K.part, K.nblk, K.m_max, K.sums,
                       (const double*)K.scal, 0);
  hipLaunchKernelGGL(k_orth<KM>, g, dim3(KT), 0, s, b.dm, Vc, k, (double2*)w, K.m_max, fold, (const double*)K.part,
                     (const double*)K.sums, K.part2, (double2*)K.H, K.scal);
  if (!fold)
    hipLaunchKernelGGL(k_kry_fold, dim3(nv, b.ni), dim3(NT), 0, s, K.part2, K.nblk, K.m_max, K.sums,
                       (const double*)K.scal, 1);
  hipLaunchKernelGGL(k_orth_scale<KM>, dim3(nblocks(b.mx.NE * b.mx.n, KT, 2048), b.ni), dim3(KT), 0, s, b.dm, Vc, k,
                     (double2*)w, K.m_max, fold, K.nblk, (const double*)K.part2, (const double*)K.sums,
                     (double2*)K.H, K.scal);
}

void launch_orthogonalize(const Batch& b, double* const* V, int k, double* w, Krylov& K, hipStream_t s) {
  if (k + 1 <= 4) orthogonalize<4>(b, V, k, w, K, s);
  else if (k + 1 <= 8) orthogonalize<8>(b, V, k, w, K, s);
  else if (k + 1 <= 13) orthogonalize<13>(b, V, k, w, K, s);
  else orthogonalize<KMAX>(b, V, k, w, K, s);
}

// Workgroups of the passes over a Krylov vector of `total` elements, and
// whether their partial sums are folded by the launch that needs them: one
// short vector (up to four elements per thread of 256 workgroups).  Long
// vectors: enough workgroups to keep the memory system busy, about 4096 over a
// batch.
void krylov_grid(int64_t total, int ni, int* nblk, int* fold) {
  *fold = ni == 1 && total <= (int64_t)4 * 256 * KT;
  int64_t nb = std::min<int64_t>(*fold ? 256 : 2048, std::max<int64_t>(1, (total + KT - 1) / KT));
  if (ni > 1) nb = std::min<int64_t>(nb, std::max<int64_t>(8, 4096 / ni));
  *nblk = (int)nb;
}

__global__ void __launch_bounds__(KT) k_norm_part(const DevMesh* __restrict__ dm, const double2* __restrict__ x,
                                                  int m_max, double* __restrict__ part) {
  INSTANCE;
  __shared__ double lds[KT / 64];
  const int n = d.n;
  const int64_t total = d.NE * n, o = d.oE * n;
  double s = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * KT + threadIdx.x; e < total; e += (int64_t)gridDim.x * KT) {
    const double2 v = ldg2(x, o + e);
    s += gbl(d.m)[row_of(e, n)] * (v.x * v.x + v.y * v.y);
  }
  const double c = kry_sum(s, lds);
  if (threadIdx.x == 0) part[blockIdx.y * kpart_stride(gridDim.x, m_max) + blockIdx.x] = c;
}

// V_0 = phi / |phi| from the norm's partials (folded by every workgroup);
// workgroup 0 clears H and files the scalars.
__global__ void __launch_bounds__(KT) k_krylov_start(const DevMesh* __restrict__ dm, const double2* __restrict__ phi,
                                                     double2* __restrict__ v0, const double* __restrict__ part,
                                                     int nblk, int m, double* __restrict__ scal,
                                                     double2* __restrict__ H, int m_max) {
  INSTANCE;
  __shared__ double lds[KT / 64];
  const int i = blockIdx.y;
  const int64_t total = d.NE * d.n, o = d.oE * d.n;
  part += i * kpart_stride(nblk, m_max);
  double s = 0.0;
  for (int b = threadIdx.x; b < nblk; b += KT) s += part[b];
  const double beta = sqrt(kry_sum(s, lds));
  const double ib = beta > 0.0 ? 1.0 / beta : 0.0;
  if (blockIdx.x == 0) {
    H += (int64_t)i * (m_max + 1) * m_max;
    for (int t = threadIdx.x; t < (m_max + 1) * m_max; t += KT) H[t] = make_double2(0.0, 0.0);
    if (threadIdx.x == 0) {
      scal += 8 * i;
      scal[0] = beta;
      scal[4] = m;
      scal[3] = 0.0;
    }
  }
  for (int64_t e = (int64_t)blockIdx.x * KT + threadIdx.x; e < total; e += (int64_t)gridDim.x * KT)
    v0[o + e] = cscale(ib, ldg2(phi, o + e));
}

void launch_krylov_start(const Batch& b, const double* phi, double* v0, Krylov& K, int m, hipStream_t s) {
  hipLaunchKernelGGL(k_norm_part, dim3(K.nblk, b.ni), dim3(KT), 0, s, b.dm, (const double2*)phi, K.m_max, K.part);
  hipLaunchKernelGGL(k_krylov_start, dim3(nblocks(b.mx.NE * b.mx.n, KT, 2048), b.ni), dim3(KT), 0, s, b.dm,
                     (const double2*)phi, (double2*)v0, (const double*)K.part, K.nblk, m, K.scal, (double2*)K.H,
                     K.m_max);
}

// T <- exp(A) of an m x m matrix in LDS (row-major, m <= M) by the whole
// workgroup: scaling and squaring with a degree-18 Taylor polynomial at
// |A / 2^s|_1 <= 1/2 (remainder below 1e-22), the polynomial in blocks of four
// powers (Paterson and Stockmeyer 1973: seven products instead of seventeen).
// A is overwritten; on return T holds the result.  The chain of products is a
// latency: one element per thread, two barriers each.
template <int M>
struct ExpmLds {
  double2 A[M * M], B[M * M], C[M * M], D[M * M], T[M * M], S[M * M];
  int s;
};
template <int M>
__device__ __forceinline__ void expm_lds(ExpmLds<M>& L, int m) {
  const int mm = m * m, nt = (int)blockDim.x;
  auto product = [&](const double2* X, const double2* Y, int e) {
    const int i = e / m, j = e - i * m;
    double2 acc = make_double2(0.0, 0.0);
    for (int l = 0; l < m; ++l) acc = cadd(acc, cmul(X[i * m + l], Y[l * m + j]));
    return acc;
  };
  __syncthreads();
  if (threadIdx.x < 64) {  // 1-norm and scaling, a column per lane
    double c = 0.0;
    if ((int)threadIdx.x < m)
      for (int i = 0; i < m; ++i) {
        const double2 a = L.A[i * m + threadIdx.x];
        c += sqrt(a.x * a.x + a.y * a.y);
      }
    for (int o = 32; o > 0; o >>= 1) c = fmax(c, __shfl_xor(c, o, 64));
    int s = 0;
    while (c > 0.5 && s < 60) { c *= 0.5; ++s; }
    if (threadIdx.x == 0) L.s = s;
  }
  __syncthreads();
  const int s = L.s;
  const double f = ldexp(1.0, -s);
  for (int e = threadIdx.x; e < mm; e += nt) L.A[e] = cscale(f, L.A[e]);
  __syncthreads();
  for (int e = threadIdx.x; e < mm; e += nt) L.B[e] = product(L.A, L.A, e);
  __syncthreads();
  for (int e = threadIdx.x; e < mm; e += nt) {
    L.C[e] = product(L.B, L.A, e);
    L.D[e] = product(L.B, L.B, e);
  }
  __syncthreads();
  // 1 / k!, k = 0..18
  constexpr double c[19] = {1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320,
                            1.0 / 362880, 1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600, 1.0 / 6227020800.0,
                            1.0 / 87178291200.0, 1.0 / 1307674368000.0, 1.0 / 20922789888000.0,
                            1.0 / 355687428096000.0, 1.0 / 6402373705728000.0};
  for (int e = threadIdx.x; e < mm; e += nt) {
    double2 t = cadd(cscale(c[17], L.A[e]), cscale(c[18], L.B[e]));
    if (e % (m + 1) == 0) t.x += c[16];
    L.T[e] = t;
  }
  __syncthreads();
  double2* T = L.T;
  double2* S = L.S;
#pragma unroll
  for (int k = 12; k >= 0; k -= 4) {
    for (int e = threadIdx.x; e < mm; e += nt) {
      double2 t = cadd(cadd(cscale(c[k + 1], L.A[e]), cscale(c[k + 2], L.B[e])), cscale(c[k + 3], L.C[e]));
      if (e % (m + 1) == 0) t.x += c[k];
      S[e] = cadd(t, product(T, L.D, e));
    }
    __syncthreads();
    double2* x = T;
    T = S;
    S = x;
  }
  for (int q = 0; q < s; ++q) {
    for (int e = threadIdx.x; e < mm; e += nt) S[e] = product(T, T, e);
    __syncthreads();
    double2* x = T;
    T = S;
    S = x;
  }
  if (T != L.T) {
    for (int e = threadIdx.x; e < mm; e += nt) L.T[e] = T[e];
    __syncthreads();
  }
}

// y = beta expm(A) e1, A = -i tau H_m (m = scal[4]).  One workgroup per instance.
// m_try > 0 (adaptive dimension): only the error estimate of dimension m_try,
// beta h_{m_try+1,m_try} |e_{m_try}^T expm(A_{m_try}) e1|; where it is at or
// below tol the instance's dimension scal[4] becomes m_try (instances whose
// space already ended, by breakdown or an earlier estimate, are left alone).
// Measured: m = 12, 19-35 -> 12 us
__global__ void __launch_bounds__(NT) k_expm(const double2* __restrict__ H, int m_max, double tau_re, double tau_im,
                                             double* __restrict__ scal, double2* __restrict__ y, int m_try,
                                             double tol) {
  __shared__ ExpmLds<KMAX - 1> L;
  const int inst = blockIdx.y;
  H += (int64_t)inst * (m_max + 1) * m_max;
  scal += 8 * inst;
  y += (int64_t)inst * m_max;
  if (m_try > 0 && (int)scal[4] <= m_try) return;  // uniform over the workgroup
  const int m = m_try > 0 ? m_try : (int)scal[4];
  // A = -i tau H = (tau_im - i tau_re) H
  const double2 f = make_double2(tau_im, -tau_re);
  for (int e = threadIdx.x; e < m * m; e += NT) {
    const int i = e / m, j = e - i * m;
    L.A[e] = cmul(f, H[i + (int64_t)(m_max + 1) * j]);
  }
  expm_lds(L, m);
  const double beta = scal[0];
  const double2 hlast = H[m + (int64_t)(m_max + 1) * (m - 1)], ylast = L.T[(m - 1) * m];
  const double err = beta * hypot(hlast.x, hlast.y) * hypot(ylast.x, ylast.y);
  if (m_try > 0) {
    if (threadIdx.x == 0 && err <= tol) scal[4] = m;
    return;
  }
  for (int i = threadIdx.x; i < m_max; i += NT) y[i] = (i < m) ? cscale(beta, L.T[i * m]) : make_double2(0.0, 0.0);
  if (threadIdx.x == 0) scal[3] = err;
}

void launch_expm(int ni, Krylov& K, double tau_re, double tau_im, hipStream_t s) {
  hipLaunchKernelGGL(k_expm, dim3(1, ni), dim3(NT), 0, s, (const double2*)K.H, K.m_max, tau_re, tau_im, K.scal,
                     (double2*)K.y, 0, 0.0);
}

void launch_krylov_check(int ni, Krylov& K, double tau_re, double tau_im, int m_try, double tol, hipStream_t s) {
  hipLaunchKernelGGL(k_expm, dim3(1, ni), dim3(NT), 0, s, (const double2*)K.H, K.m_max, tau_re, tau_im, K.scal,
                     (double2*)K.y, m_try, tol);
}

__global__ void __launch_bounds__(NT) k_combine(const DevMesh* __restrict__ dm, const double2* const* __restrict__ V,
                                                int m, int m_max, double2* __restrict__ phi,
                                                const double2* __restrict__ y) {
  INSTANCE;
  const int64_t total = d.NE * d.n, o = d.oE * d.n;
  y += (int64_t)blockIdx.y * m_max;
  double2 yy[KMAX];
#pragma unroll
  for (int j = 0; j < KMAX; ++j) yy[j] = (j < m) ? y[j] : make_double2(0.0, 0.0);
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < total; e += (int64_t)gridDim.x * NT) {
    double2 s = make_double2(0.0, 0.0);
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
      if (j < m) s = cadd(s, cmul(yy[j], ldg2(V[j], o + e)));
    phi[o + e] = s;
  }
}

void launch_combine(const Batch& b, double* const* V, int m, double* phi, Krylov& K, hipStream_t s) {
  hipLaunchKernelGGL(k_combine, dim3(nblocks(b.mx.NE * b.mx.n, NT, 8192), b.ni), dim3(NT), 0, s, b.dm,
                     (const double2* const*)V, m, K.m_max, (double2*)phi, (const double2*)K.y);
}

// =====================================================================
// Poisson: moments, boundary values, right-hand side.  Column c of the n^2
// real columns is (r, s, part) = colinfo[c].
// =====================================================================
constexpr int MP_CH = 32;

__device__ __forceinline__ double pair_density(const double2* phi, int n, int64_t i, int r, int s, int part) {
  double2 a = phi[i * n + r], b = phi[i * n + s];
  // conj(a) b
  return part == 0 ? (a.x * b.x + a.y * b.y) : (a.x * b.y - a.y * b.x);
}

// Multipole moments Q[t][c] = sum_i R_t(x_i) m_i rho_c(x_i) of the pair
// densities, per instance, with register tiles: each thread accumulates a
// tile of MT_H harmonics x MT_C columns, so every pair of LDS reads (one
// harmonic quadruple, one column quadruple) feeds 16 FMAs.  Tiles are
// numbered column-tile fastest; grid.z splits the tiles in sets of NT.
constexpr int MT_H = 4, MT_C = 4;
constexpr int MP_HP = 172;  // harmonics padded to a multiple of MT_H
__global__ void __launch_bounds__(NT) k_moments_rb(const DevMesh* __restrict__ dm, const double2* __restrict__ phi,
                                                   int lmax, int ncol, const int* __restrict__ colinfo,
                                                   double* __restrict__ part) {
  INSTANCE;
  __shared__ double sR[MP_CH * MP_HP];
  __shared__ double sW[MP_CH * 64];
  const int nh = (lmax + 1) * (lmax + 1);
  const int nhp = (nh + MT_H - 1) / MT_H * MT_H;
  const int ncp = (ncol + MT_C - 1) / MT_C * MT_C;
  const int nout = nh * ncol;
  const int n = d.n;
  phi += d.oE * n;
  const double cx = d.center[0], cy = d.center[1], cz = d.center[2];
  const int tiles_c = ncp / MT_C, tiles = (nhp / MT_H) * tiles_c;
  const int tile = blockIdx.z * NT + threadIdx.x;
  const bool act = tile < tiles;
  const int t0 = act ? (tile / tiles_c) * MT_H : 0, c0 = act ? (tile % tiles_c) * MT_C : 0;
  double acc[MT_H][MT_C];
#pragma unroll
  for (int a = 0; a < MT_H; ++a)
#pragma unroll
    for (int b = 0; b < MT_C; ++b) acc[a][b] = 0.0;
  const int64_t rows = d.NE;
  for (int64_t base = (int64_t)blockIdx.x * MP_CH; base < rows; base += (int64_t)gridDim.x * MP_CH) {
    const int cnt = (int)((rows - base) < MP_CH ? (rows - base) : MP_CH);
    __syncthreads();
    // harmonics of the chunk's rows, one (row, order m) per thread; padding zero
    for (int w = threadIdx.x; w < MP_CH * (lmax + 1); w += NT) {
      const int r = w / (lmax + 1), m = w - r * (lmax + 1);
      double* R = sR + r * nhp;
      if (r < cnt) {
        const int64_t i = base + r;
        solid_regular_m(d.xyz[3 * i] - cx, d.xyz[3 * i + 1] - cy, d.xyz[3 * i + 2] - cz, lmax, m, R);
      } else {
        for (int l = m; l <= lmax; ++l) {
          R[l * l + m] = 0.0;
          if (m > 0) R[l * l + l + m] = 0.0;
        }
      }
    }
    if (nhp > nh)
      for (int e = threadIdx.x; e < MP_CH * (nhp - nh); e += NT) sR[(e / (nhp - nh)) * nhp + nh + e % (nhp - nh)] = 0.0;
    for (int e = threadIdx.x; e < MP_CH * ncp; e += NT) {
      const int r = e / ncp, c = e - r * ncp;
      double v = 0.0;
      if (r < cnt && c < ncol) {
        const int64_t i = base + r;
        const int ci = colinfo[c];
        v = d.m[i] * pair_density(phi, n, i, ci & 255, (ci >> 8) & 255, ci >> 16);
      }
      sW[r * ncp + c] = v;
    }
    __syncthreads();
    if (act)
      for (int r = 0; r < cnt; ++r) {
        double hv[MT_H], wv[MT_C];
#pragma unroll
        for (int a = 0; a < MT_H; ++a) hv[a] = sR[r * nhp + t0 + a];
#pragma unroll
        for (int b = 0; b < MT_C; ++b) wv[b] = sW[r * ncp + c0 + b];
#pragma unroll
        for (int a = 0; a < MT_H; ++a)
#pragma unroll
          for (int b = 0; b < MT_C; ++b) acc[a][b] += hv[a] * wv[b];
      }
  }
  if (!act) return;
  double* pb = part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * nout;
#pragma unroll
  for (int a = 0; a < MT_H; ++a)
#pragma unroll
    for (int b = 0; b < MT_C; ++b)
      if (t0 + a < nh && c0 + b < ncol) pb[(t0 + a) * ncol + c0 + b] = acc[a][b];
}
// The same moments on the matrix cores (16 or more columns): per chunk of
// MP_CH rows the harmonics R[row][h] and the weighted pair densities
// W[row][c] are staged in LDS once, and Q[h][c] += sum over rows of
// R[row][h] W[row][c] accumulates in FP64 MFMA tiles of 16 harmonics x 16
// columns, four rows per instruction.  The (harmonic tile, column tile)
// pairs are dealt round-robin to the four waves, at most MM_TW per wave.
// Lane layout of v_mfma_f64_16x16x4_f64 (measured): A[i][k] from lane 16 k + i,
// B[k][j] from lane 16 k + j, and accumulator v of lane l holds
// D[4 v + l / 16][l % 16].
constexpr int MM_HP = 176;  // harmonics padded to a multiple of 16 (lmax <= 12: 169)
constexpr int MM_TW = 11;   // 11 harmonic tiles x 4 column tiles over 4 waves
constexpr int MM_CH = 16;   // rows per chunk (30.5 KB of LDS: five workgroups per compute unit)
typedef double dvec4_t __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(NT) k_moments_mfma(const DevMesh* __restrict__ dm, const double2* __restrict__ phi,
                                                     int lmax, int ncol, const int* __restrict__ colinfo,
                                                     double* __restrict__ part) {
  INSTANCE;
  __shared__ double sR[MM_CH * MM_HP];
  __shared__ double sW[MM_CH * 64];
  const int nh = (lmax + 1) * (lmax + 1);
  const int nct = (ncol + 15) / 16, ntile = ((nh + 15) / 16) * nct;
  const int nout = nh * ncol;
  const int n = d.n;
  phi += d.oE * n;
  const double cx = d.center[0], cy = d.center[1], cz = d.center[2];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  dvec4_t acc[MM_TW];
#pragma unroll
  for (int j = 0; j < MM_TW; ++j) acc[j] = dvec4_t{0.0, 0.0, 0.0, 0.0};
  const int64_t rows = d.NE;
  for (int64_t base = (int64_t)blockIdx.x * MM_CH; base < rows; base += (int64_t)gridDim.x * MM_CH) {
    const int cnt = (int)((rows - base) < MM_CH ? (rows - base) : MM_CH);
    __syncthreads();
    for (int w = threadIdx.x; w < MM_CH * (lmax + 1); w += NT) {
      const int r = w / (lmax + 1), m = w - r * (lmax + 1);
      double* R = sR + r * MM_HP;
      if (r < cnt) {
        const int64_t i = base + r;
        solid_regular_m(d.xyz[3 * i] - cx, d.xyz[3 * i + 1] - cy, d.xyz[3 * i + 2] - cz, lmax, m, R);
      } else {
        for (int l = m; l <= lmax; ++l) {
          R[l * l + m] = 0.0;
          if (m > 0) R[l * l + l + m] = 0.0;
        }
      }
    }
    for (int e = threadIdx.x; e < MM_CH * (MM_HP - nh); e += NT)
      sR[(e / (MM_HP - nh)) * MM_HP + nh + e % (MM_HP - nh)] = 0.0;
    for (int e = threadIdx.x; e < MM_CH * 64; e += NT) {
      const int r = e >> 6, c = e & 63;
      double v = 0.0;
      if (r < cnt && c < ncol) {
        const int64_t i = base + r;
        const int ci = colinfo[c];
        v = d.m[i] * pair_density(phi, n, i, ci & 255, (ci >> 8) & 255, ci >> 16);
      }
      sW[e] = v;
    }
    __syncthreads();
#pragma unroll
    for (int k0 = 0; k0 < MM_CH; k0 += 4) {
      const int kr = k0 + (lane >> 4), li = lane & 15;
#pragma unroll
      for (int j = 0; j < MM_TW; ++j) {
        const int tile = wave + 4 * j;
        if (tile < ntile) {
          const int t = tile / nct, u = tile - t * nct;
          const double a = sR[kr * MM_HP + 16 * t + li];
          const double b = sW[kr * 64 + 16 * u + li];
          acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[j], 0, 0, 0);
        }
      }
    }
  }
  double* pb = part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * nout;
#pragma unroll
  for (int j = 0; j < MM_TW; ++j) {
    const int tile = wave + 4 * j;
    if (tile >= ntile) continue;
    const int t = tile / nct, u = tile - t * nct;
    const int c = 16 * u + (lane & 15);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int h = 16 * t + 4 * v + (lane >> 4);
      if (h < nh && c < ncol) pb[h * ncol + c] = acc[j][v];
    }
  }
}

// W[NE + b][c] = sum_t table[b][t] Q[t][c]
__global__ void k_bnd_eval(const DevMesh* __restrict__ dm, int nh, const double* __restrict__ Q, int ncol,
                           double* __restrict__ W) {
  INSTANCE;
  const int64_t total = d.Nb * ncol;
  Q += (int64_t)blockIdx.y * nh * ncol;
  W += d.oF * ncol;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < total; e += (int64_t)gridDim.x * NT) {
    int64_t b = e / ncol;
    int c = (int)(e - b * ncol);
    double s = 0.0;
    for (int t = 0; t < nh; ++t) s += d.bnd_table[b * nh + t] * Q[t * ncol + c];
    W[(d.NE + b) * ncol + c] = s;
  }
}

// Boundary lift through the element stiffness: acc += K_full x over the
// listed boundary cells, with x the lift (boundary rows and the boundary-
// master share of hanging rows; DoF rows read as zero).  x over full rows,
// acc over extended rows; boundary rows of acc are skipped.
template <int P>
__global__ void __launch_bounds__(NT) k_lift_poisson(const DevMesh* __restrict__ dm, const double* __restrict__ x,
                                                     double* __restrict__ acc, int ncol) {
  INSTANCE;
  constexpr int P3 = P * P * P;
  __shared__ double sx[P3 * 64];
  __shared__ int snode[P3];
  x += d.oF * ncol;
  acc += d.oE * ncol;
  for (int64_t cb = blockIdx.x; cb < d.n_bnd_cells; cb += gridDim.x) {
    const int64_t e = d.bnd_cells[cb];
    __syncthreads();
    for (int t = threadIdx.x; t < P3; t += NT) snode[t] = d.cell_nodes[e * P3 + t];
    __syncthreads();
    for (int idx = threadIdx.x; idx < P3 * ncol; idx += NT) {
      int t = idx / ncol, c = idx - t * ncol;
      int node = snode[t];
      double v = 0.0;
      if (node >= d.NE) {
        v = x[(int64_t)node * ncol + c];
      } else if (node >= d.N) {
        int64_t h = node - d.N;
        for (int k = d.hang_ptr[h]; k < d.hang_ptr[h + 1]; ++k)
          if (d.hang_col[k] >= d.NE) v += d.hang_w[k] * x[(int64_t)d.hang_col[k] * ncol + c];
      }
      sx[c * P3 + t] = v;
    }
    __syncthreads();
    const double hh = d.cell_hh[e];
    for (int idx = threadIdx.x; idx < P3 * ncol; idx += NT) {
      int t = idx / ncol, c = idx - t * ncol;
      int node = snode[t];
      if (node >= d.NE) continue;
      int a = t % P, b = (t / P) % P, cc = t / (P * P);
      const double* xo = sx + c * P3;
      double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
      for (int q = 0; q < P; ++q) {
        s0 += d.A[a * P + q] * xo[(cc * P + b) * P + q];
        s1 += d.A[b * P + q] * xo[(cc * P + q) * P + a];
        s2 += d.A[cc * P + q] * xo[(q * P + b) * P + a];
      }
      double y = hh * (d.w[b] * d.w[cc] * s0 + d.w[a] * d.w[cc] * s1 + d.w[a] * d.w[b] * s2);
      atomicAdd(acc + (int64_t)node * ncol + c, y);
    }
  }
}

static void launch_lift_poisson(const Batch& b, const double* x, double* acc, int ncol, hipStream_t s) {
  const int64_t ncell = b.mx.n_bnd_cells;
  if (ncell == 0) return;
  const dim3 g((unsigned)(ncell < 65536 ? ncell : 65536), b.ni);
  switch (b.mx.P) {
    case 2: hipLaunchKernelGGL(k_lift_poisson<2>, g, dim3(NT), 0, s, b.dm, x, acc, ncol); break;
    case 3: hipLaunchKernelGGL(k_lift_poisson<3>, g, dim3(NT), 0, s, b.dm, x, acc, ncol); break;
    default: hipLaunchKernelGGL(k_lift_poisson<4>, g, dim3(NT), 0, s, b.dm, x, acc, ncol);
  }
}

// Hanging rows of a real column array; with_bnd includes boundary masters.
__global__ void k_fill_real(const DevMesh* __restrict__ dm, double* __restrict__ x, int xfull, int ncol,
                            int with_bnd, double* __restrict__ acc) {
  INSTANCE;
  const int64_t total = d.Nh * ncol;
  x += (xfull ? d.oF : d.oE) * ncol;
  if (acc) acc += d.oE * ncol;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < total; e += (int64_t)gridDim.x * NT) {
    int64_t h = e / ncol;
    int c = (int)(e - h * ncol);
    double s = 0.0;
    for (int t = d.hang_ptr[h]; t < d.hang_ptr[h + 1]; ++t) {
      int col = d.hang_col[t];
      if (col < d.N || with_bnd) s += d.hang_w[t] * x[(int64_t)col * ncol + c];
    }
    x[(d.N + h) * ncol + c] = s;
    if (acc) acc[(d.N + h) * ncol + c] = 0.0;
  }
}

void launch_fill_real(const Batch& b, double* x, int xfull, int ncol, int with_bnd, double* acc, hipStream_t s) {
  if (b.mx.Nh == 0) return;
  hipLaunchKernelGGL(k_fill_real, dim3(nblocks(b.mx.Nh * ncol), b.ni), dim3(NT), 0, s, b.dm, x, xfull, ncol,
                     with_bnd, acc);
}

// Zero rows [lo, hi) (lo, hi: 0 = 0, 1 = N, 2 = NE) of a real column array over extended rows.
__global__ void k_zero_rows(const DevMesh* __restrict__ dm, double* __restrict__ x, int ncol, int lo, int hi) {
  INSTANCE;
  const int64_t r0 = lo == 0 ? 0 : (lo == 1 ? d.N : d.NE), r1 = hi == 0 ? 0 : (hi == 1 ? d.N : d.NE);
  x += (d.oE + r0) * ncol;
  const int64_t total = (r1 - r0) * ncol;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < total; e += (int64_t)gridDim.x * NT) x[e] = 0.0;
}

// RHS: b = 4 pi C^T (m rho) - C^T acc;  partial |b|^2 (acc DoF rows zeroed).
__global__ void __launch_bounds__(NT) k_poisson_rhs(const DevMesh* __restrict__ dm, const double2* __restrict__ phi,
                                                    double* __restrict__ acc, int ncol,
                                                    const int* __restrict__ colinfo, double* __restrict__ rhs,
                                                    int64_t part_stride, double* __restrict__ part) {
  INSTANCE;
  __shared__ double lds[NT];
  const int groups = NT / ncol;
  const int g = threadIdx.x / ncol, c = threadIdx.x - g * ncol;
  const bool act = g < groups;
  double bb = 0.0;
  const int n = d.n;
  phi += d.oE * n;
  acc += d.oE * ncol;
  rhs += d.oE * ncol;
  const int ci = colinfo[act ? c : 0];
  const int r = ci & 255, s = (ci >> 8) & 255, pr = ci >> 16;
  if (act)
    for (int64_t k = (int64_t)blockIdx.x * groups + g; k < d.N; k += (int64_t)gridDim.x * groups) {
      double f = 4.0 * M_PI * d.m[k] * pair_density(phi, n, k, r, s, pr) - acc[k * ncol + c];
      acc[k * ncol + c] = 0.0;
      int mi = d.ma_index[k];
      if (mi >= 0)
        for (int t = d.ct_ptr[mi]; t < d.ct_ptr[mi + 1]; ++t) {
          int64_t h = d.ct_row[t];
          f += d.ct_w[t] * (4.0 * M_PI * d.m[h] * pair_density(phi, n, h, r, s, pr) - acc[h * ncol + c]);
        }
      rhs[k * ncol + c] = f;
      bb += f * f;
    }
  lds[threadIdx.x] = act ? bb : 0.0;
  __syncthreads();
  if (threadIdx.x < ncol) {
    double t = 0.0;
    for (int q = 0; q < groups; ++q) t += lds[q * ncol + threadIdx.x];
    part[blockIdx.y * part_stride + (int64_t)blockIdx.x * ncol + threadIdx.x] = t;
  }
}

// sc[i][slot][c] = sum_b part[i][b][c]; one workgroup per (column, instance)
__global__ void __launch_bounds__(NT) k_col_sum(const double* __restrict__ part, int64_t part_stride, int nblk,
                                                int ncol, double* __restrict__ sc, int slot) {
  __shared__ double lds4[4];
  const int c = blockIdx.x;
  const double s = sum_partials(part + blockIdx.y * part_stride, nblk, ncol, c, lds4);
  if (threadIdx.x == 0) sc[(int64_t)blockIdx.y * SC_SLOTS * ncol + slot * ncol + c] = s;
}

static int rhs_blocks(const Batch& b, int ncol) { return nblocks(b.mx.N, NT / ncol, 1024); }

void launch_poisson_pipeline_moments(const Batch& b, const double* phi, const int* colinfo, PoissonWs& P,
                                     hipStream_t s) {
  const int nout = P.nharm * P.ncol;
  const double2* ph = (const double2*)phi;
  if (P.ncol >= 16 && P.ncol <= 64 && P.nharm <= MM_HP) {  // matrix cores: every tile in one workgroup
    hipLaunchKernelGGL(k_moments_mfma, dim3(P.mblk, b.ni), dim3(NT), 0, s, b.dm, ph, P.lmax, P.ncol, colinfo,
                       P.mpart);
  } else {
    // register tiles of 4 harmonics x 4 columns, sets of NT tiles over grid.z
    const int tiles = ((P.nharm + MT_H - 1) / MT_H) * ((P.ncol + MT_C - 1) / MT_C);
    const unsigned nz = (unsigned)((tiles + NT - 1) / NT);
    hipLaunchKernelGGL(k_moments_rb, dim3(P.mblk, b.ni, nz), dim3(NT), 0, s, b.dm, ph, P.lmax, P.ncol, colinfo,
                       P.mpart);
  }
  launch_sum_parts(P.mpart, P.mblk, nout, P.Q, b.ni, s);
}

void launch_bnd_eval(const Batch& b, PoissonWs& P, double* W, hipStream_t s) {
  if (b.mx.Nb == 0) return;
  hipLaunchKernelGGL(k_bnd_eval, dim3(nblocks(b.mx.Nb * P.ncol), b.ni), dim3(NT), 0, s, b.dm, P.nharm, P.Q, P.ncol,
                     W);
}

void launch_poisson_rhs_full(const Batch& b, const double* phi, double* W, const int* colinfo, double* rhs,
                             PoissonWs& P, hipStream_t s) {
  const int ncol = P.ncol;
  launch_zero(P.acc, b.tE * ncol, s);  // the lift pass accumulates with atomics
  launch_lift_poisson(b, W, P.acc, ncol, s);
  const int nb = rhs_blocks(b, ncol);
  hipLaunchKernelGGL(k_poisson_rhs, dim3(nb, b.ni), dim3(NT), 0, s, b.dm, (const double2*)phi, P.acc, ncol, colinfo,
                     rhs, P.part_stride, P.part);
  hipLaunchKernelGGL(k_col_sum, dim3(ncol, b.ni), dim3(NT), 0, s, P.part, P.part_stride, nb, ncol, P.sc, (int)SC_BB);
  // hanging rows of acc back to zero
  if (b.mx.Nh > 0)
    hipLaunchKernelGGL(k_zero_rows, dim3(nblocks(b.mx.Nh * ncol, NT, 4096), b.ni), dim3(NT), 0, s, b.dm, P.acc,
                       ncol, 1, 2);
}

// =====================================================================
// Small dense kernels (one workgroup per instance, work on thread 0).
// =====================================================================
// Regularised inverse of the Hermitian 1-RDM: eigen-decomposition of the
// real 2n x 2n embedding [[Re, -Im], [Im, Re]] by Jacobi rotations, d -> d +
// eps exp(-d/eps), inverse from the eigenpairs.  One wave per instance with
// the matrices in LDS.  Each sweep runs 2n - 1 rounds of n disjoint pivot
// pairs (the round-robin ordering): the pairs' angles come from the entries
// at the start of the round, then all column rotations (of A and of the
// eigenvector matrix) and all row rotations are applied at once.  Disjoint
// rotations commute, so a round is the same as those rotations in sequence.
__device__ __forceinline__ double wave_sum_xor(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);  // every lane gets the same total
  return v;
}
__global__ void __launch_bounds__(64) k_ginv(const double2* __restrict__ gamma, int n, double eps,
                                             double2* __restrict__ ginv, int* __restrict__ flag) {
  __shared__ double a[16 * 16], V[16 * 16], dinv[16];
  __shared__ double rc[8], rs[8];
  __shared__ int rp[8], rq[8];
  __shared__ int badk[16];
  const int inst = blockIdx.x, lane = threadIdx.x;
  gamma += (int64_t)inst * n * n;
  ginv += (int64_t)inst * n * n;
  const int N2 = 2 * n, npair = n, m = N2 - 1;
  for (int e = lane; e < n * n; e += 64) {
    const int i = e / n, j = e - i * n;
    // Hermitian part
    const double re = 0.5 * (gamma[i * n + j].x + gamma[j * n + i].x);
    const double im = 0.5 * (gamma[i * n + j].y - gamma[j * n + i].y);
    a[i * N2 + j] = re;
    a[(i + n) * N2 + (j + n)] = re;
    a[i * N2 + (j + n)] = -im;
    a[(i + n) * N2 + j] = im;
  }
  for (int e = lane; e < N2 * N2; e += 64) V[e] = (e / N2 == e % N2) ? 1.0 : 0.0;
  __syncthreads();
  for (int sweep = 0; sweep < 60; ++sweep) {
    double off = 0.0, tot = 0.0;
    for (int e = lane; e < N2 * N2; e += 64) {
      const double v = a[e];
      tot += v * v;
      if (e / N2 != e % N2) off += v * v;
    }
    off = wave_sum_xor(off);
    tot = wave_sum_xor(tot);
    // off-diagonal Frobenius norm at 1e-15 of the whole: above the rounding
    // floor of the rotations (about N2 eps^2 in the squares), so the sweeps stop
    // once converged instead of running to the cap on a stagnating remainder
    if (off <= 1e-30 * tot) break;
    for (int r = 0; r < m; ++r) {
      if (lane < npair) {
        // pair `lane` of round r: (N2 - 1, r) for lane 0, else (r + lane, r - lane) mod m
        int p = lane == 0 ? r : (r + lane) % m, q = lane == 0 ? N2 - 1 : (r - lane + m) % m;
        if (p > q) { const int t = p; p = q; q = t; }
        const double apq = a[p * N2 + q];
        double c = 1.0, sn = 0.0;
        if (fabs(apq) >= 1e-300) {
          const double theta = (a[q * N2 + q] - a[p * N2 + p]) / (2.0 * apq);
          const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
          c = 1.0 / sqrt(t * t + 1.0);
          sn = t * c;
        }
        rp[lane] = p;
        rq[lane] = q;
        rc[lane] = c;
        rs[lane] = sn;
      }
      __syncthreads();
      for (int w = lane; w < npair * N2; w += 64) {  // columns p, q of a and V
        const int k = w / N2, i = w - k * N2;
        const int p = rp[k], q = rq[k];
        const double c = rc[k], sn = rs[k];
        const double aip = a[i * N2 + p], aiq = a[i * N2 + q];
        a[i * N2 + p] = c * aip - sn * aiq;
        a[i * N2 + q] = sn * aip + c * aiq;
        const double vip = V[i * N2 + p], viq = V[i * N2 + q];
        V[i * N2 + p] = c * vip - sn * viq;
        V[i * N2 + q] = sn * vip + c * viq;
      }
      __syncthreads();
      for (int w = lane; w < npair * N2; w += 64) {  // rows p, q of a
        const int k = w / N2, j = w - k * N2;
        const int p = rp[k], q = rq[k];
        const double c = rc[k], sn = rs[k];
        const double apj = a[p * N2 + j], aqj = a[q * N2 + j];
        a[p * N2 + j] = c * apj - sn * aqj;
        a[q * N2 + j] = sn * apj + c * aqj;
      }
      __syncthreads();
    }
  }
  if (lane < N2) {
    const double dk = a[lane * N2 + lane];
    const double dr = dk + eps * exp(-dk / eps);
    badk[lane] = (!(dr > 0.0) || !isfinite(dr)) ? 1 : 0;
    dinv[lane] = 1.0 / dr;
  }
  __syncthreads();
  for (int e = lane; e < n * n; e += 64) {
    const int i = e / n, j = e - i * n;
    double re = 0.0, im = 0.0;
    for (int k = 0; k < N2; ++k) {
      re += V[i * N2 + k] * dinv[k] * V[j * N2 + k];
      im += V[(i + n) * N2 + k] * dinv[k] * V[j * N2 + k];
    }
    ginv[i * n + j] = make_double2(re, im);
  }
  if (lane == 0) {
    int bad = 0;
    for (int k = 0; k < N2; ++k) bad |= badk[k];
    flag[inst] = bad;
  }
}

void launch_ginv(int ni, const double* gamma, int n, double eps, double* ginv, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_ginv, dim3(ni), dim3(64), 0, s, (const double2*)gamma, n, eps, (double2*)ginv, flag);
}

// out[i]: [0] energy, [1] dipole, [2] max |S - I|, [3] kinetic momentum along
// e (sum gamma_pq <phi_p|-i S_e|phi_q>, plus N A in the velocity gauge)
__global__ void __launch_bounds__(NT) k_observe(const DevMesh* __restrict__ dm, const double2* __restrict__ gamma,
                                                const double2* __restrict__ Gamma, const double2* __restrict__ h,
                                                const double2* __restrict__ g, const double2* __restrict__ z,
                                                const double2* __restrict__ S, const double2* __restrict__ pm,
                                                const double* __restrict__ Ef, double* __restrict__ out) {
  __shared__ double lds4[4];
  const int inst = blockIdx.x;
  const DevMesh& d = dm[inst];
  const int n = d.n, nn = n * n;
  gamma += (int64_t)inst * nn;
  Gamma += (int64_t)inst * nn * nn;
  h += (int64_t)inst * nn;
  g += (int64_t)inst * nn * nn;
  z += (int64_t)inst * nn;
  S += (int64_t)inst * nn;
  pm += (int64_t)inst * nn;
  out += 8 * inst;
  // Re sum h gamma, Re sum gamma z, Re sum gamma p, tr gamma and Re sum g Gamma over the block
  double e1 = 0.0, e2 = 0.0, dip = 0.0, mom = 0.0, tr = 0.0;
  for (int i = threadIdx.x; i < nn; i += NT) {
    e1 += h[i].x * gamma[i].x - h[i].y * gamma[i].y;
    dip += gamma[i].x * z[i].x - gamma[i].y * z[i].y;
    mom += gamma[i].x * pm[i].x - gamma[i].y * pm[i].y;
    if (i % (n + 1) == 0) tr += gamma[i].x;
  }
  for (int i = threadIdx.x; i < nn * nn; i += NT) e2 += g[i].x * Gamma[i].x - g[i].y * Gamma[i].y;
  e1 = block_sum_all(e1, lds4);
  e2 = block_sum_all(e2, lds4);
  dip = block_sum_all(dip, lds4);
  mom = block_sum_all(mom, lds4);
  tr = block_sum_all(tr, lds4);
  if (threadIdx.x != 0) return;
  double orth = 0.0;
  for (int i = 0; i < nn; ++i) {
    const int p = i / n, q = i % n;
    const double dx = S[i].x - (p == q ? 1.0 : 0.0);
    orth = fmax(orth, hypot(dx, S[i].y));
  }
  out[0] = e1 + 0.5 * e2 + d.vnn;
  out[1] = dip;
  out[2] = orth;
  out[3] = mom + (d.gauge == 1 ? tr * Ef[0] * d.E0 : 0.0);
}

void launch_observe(const Batch& b, const double* gamma, const double* Gamma, const double* h, const double* g,
                    const double* zmat, const double* S, const double* pmat, const double* Ef, double* out,
                    hipStream_t s) {
  hipLaunchKernelGGL(k_observe, dim3(b.ni), dim3(NT), 0, s, b.dm, (const double2*)gamma, (const double2*)Gamma,
                     (const double2*)h, (const double2*)g, (const double2*)zmat, (const double2*)S,
                     (const double2*)pmat, Ef, out);
}

// Gram-Schmidt in M as x <- x R^-1 with S = R^H R (Cholesky), R upper.
__global__ void k_chol_inv(const double2* __restrict__ S, int n, double2* __restrict__ Rinv) {
  if (threadIdx.x != 0) return;
  S += (int64_t)blockIdx.x * n * n;
  Rinv += (int64_t)blockIdx.x * n * n;
  double2 R[64], Ri[64];
  for (int i = 0; i < n * n; ++i) { R[i] = make_double2(0, 0); Ri[i] = make_double2(0, 0); }
  for (int j = 0; j < n; ++j) {
    // R_jj = sqrt(S_jj - sum_k |R_kj|^2); R_ji = (S_ji - sum_k conj(R_kj) R_ki) / R_jj
    double dd = S[j * n + j].x;
    for (int k = 0; k < j; ++k) dd -= R[k * n + j].x * R[k * n + j].x + R[k * n + j].y * R[k * n + j].y;
    double rjj = sqrt(fmax(dd, 1e-300));
    R[j * n + j] = make_double2(rjj, 0.0);
    for (int i = j + 1; i < n; ++i) {
      double2 s = S[j * n + i];
      for (int k = 0; k < j; ++k) s = csub(s, cjmul(R[k * n + j], R[k * n + i]));
      R[j * n + i] = cscale(1.0 / rjj, s);
    }
  }
  // invert upper triangular R
  for (int i = n - 1; i >= 0; --i) {
    Ri[i * n + i] = make_double2(1.0 / R[i * n + i].x, 0.0);
    for (int j = i + 1; j < n; ++j) {
      double2 s = make_double2(0, 0);
      for (int k = i + 1; k <= j; ++k) s = cadd(s, cmul(R[i * n + k], Ri[k * n + j]));
      Ri[i * n + j] = cscale(-1.0 / R[i * n + i].x, s);
    }
  }
  for (int i = 0; i < n * n; ++i) Rinv[i] = Ri[i];
}

__global__ void k_right_mul(const DevMesh* __restrict__ dm, double2* __restrict__ x, const double2* __restrict__ Ri) {
  INSTANCE;
  const int n = d.n;
  x += d.oE * n;
  Ri += (int64_t)blockIdx.y * n * n;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < d.NE; i += (int64_t)gridDim.x * NT) {
    double2 row[8], out[8];
    for (int p = 0; p < n; ++p) row[p] = x[i * n + p];
    for (int q = 0; q < n; ++q) {
      double2 s = make_double2(0, 0);
      for (int p = 0; p <= q; ++p) s = cadd(s, cmul(row[p], Ri[p * n + q]));
      out[q] = s;
    }
    for (int q = 0; q < n; ++q) x[i * n + q] = out[q];
  }
}

void launch_orthonormalize_full(const Batch& b, const double* S, double* Rinv, double* x, hipStream_t s) {
  hipLaunchKernelGGL(k_chol_inv, dim3(b.ni), dim3(64), 0, s, (const double2*)S, b.mx.n, (double2*)Rinv);
  hipLaunchKernelGGL(k_right_mul, dim3(nblocks(b.mx.NE, NT, 4096), b.ni), dim3(NT), 0, s, b.dm, (double2*)x,
                     (const double2*)Rinv);
}

// =====================================================================
// CI: excitation-table sigma vector, RDMs, Lanczos in one workgroup per
// instance.  Tables: ex[J][p*n+q] = I | (sign<0) << 30 with E_pq |I> =
// sign |J>, or -1.  Vectors of instance i at offset i * dim.
// =====================================================================
// (E_pq C)(J): the alpha and the beta excitation that lead to determinant J.
__device__ __forceinline__ double2 ci_excited(const CIDev& c, const double2* __restrict__ C, int J, int pq) {
  const int nn = c.n * c.n, Ja = J / c.NB, Jb = J - Ja * c.NB;
  const int ta = gbl(c.exa)[Ja * nn + pq], tb = gbl(c.exb)[Jb * nn + pq];
  double2 s = make_double2(0.0, 0.0);
  if (ta >= 0) s = cscale((ta >> 30) ? -1.0 : 1.0, C[(ta & 0x3fffffff) * c.NB + Jb]);
  if (tb >= 0) s = cadd(s, cscale((tb >> 30) ? -1.0 : 1.0, C[Ja * c.NB + (tb & 0x3fffffff)]));
  return s;
}

// The excited amplitudes (E_pq C)(J) of CI_R determinants from J0 on into LDS
// (real and imaginary parts, row r = J - J0, zero past the ends), by 256 threads:
// one to four per thread, their table entries and then their amplitudes
// requested together.
constexpr int CI_R = 16, CI_LD = 80;
__device__ __forceinline__ void ci_fill(const CIDev& c, const double2* __restrict__ C, int J0, double* re, double* im) {
  const int nn = c.n * c.n, w = (nn + 15) / 16 * 16;   // padded pairs: 16 w values, w / 16 per thread
  int ta[4], tb[4], ia[4], ib[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    ta[j] = tb[j] = -1;
    ia[j] = ib[j] = 0;
    const int e = threadIdx.x + NT * j, r = e / w, pq = e - r * w, J = J0 + r;
    if (r < CI_R && J < c.dim && pq < nn) {
      const int Ja = J / c.NB, Jb = J - Ja * c.NB;
      ta[j] = gbl(c.exa)[Ja * nn + pq];
      tb[j] = gbl(c.exb)[Jb * nn + pq];
      ia[j] = Jb;
      ib[j] = Ja * c.NB;
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = threadIdx.x + NT * j, r = e / w, pq = e - r * w;
    double2 va = make_double2(0.0, 0.0), vb = va;
    if (ta[j] >= 0) va = ldg2(C, (ta[j] & 0x3fffffff) * c.NB + ia[j]);
    if (tb[j] >= 0) vb = ldg2(C, ib[j] + (tb[j] & 0x3fffffff));
    const double fa = (ta[j] >> 30) & 1 ? -1.0 : 1.0, fb = (tb[j] >> 30) & 1 ? -1.0 : 1.0;
    if (r < CI_R) {
      re[r * CI_LD + pq] = fa * va.x + fb * vb.x;
      im[r * CI_LD + pq] = fa * va.y + fb * vb.y;
    }
  }
}

// Transition RDMs gamma_pq = <A|E_pq|B>, Gamma[p][q][r][s] = <A|E_pq E_rs|B>
// - delta_qr gamma_ps, from G = (E_qp A)^H (E_rs B) over the determinants (A = B:
// the RDMs).  A workgroup takes chunks of CI_R determinants: their excited
// amplitudes go straight to LDS, and G accumulates in FP64 matrix-core tiles of
// 16 x 16 pairs (lane layout of k_moments_mfma).  One workgroup for a small
// space (the result is final), else up to 128 with partial sums that
// k_ci_rdm_finish adds up, neighbouring lanes on neighbouring pairs.
// Measured, against a table of excited amplitudes in memory, two Gram passes with
// a strided sum each and the assembly (six launches): 54 -> 20 us at CAS(10e, 8o)
// (3,136 determinants, 64 pairs)
// NTL: tiles of 16 pairs; a wave's last tiles past the end repeat the last one
// and are not stored, so the matrix instructions need no branch (with one, the
// compiler moves the accumulators around it).
constexpr int CI_BLK = 128;
template <int NTL>
__global__ void __launch_bounds__(NT) k_ci_rdm(CIDev c, const double2* __restrict__ A, const double2* __restrict__ B,
                                               int same, double2* __restrict__ part, double2* __restrict__ gamma,
                                               double2* __restrict__ Gamma) {
  typedef double dvec4c_t __attribute__((ext_vector_type(4)));
  __shared__ double sar[CI_R * CI_LD], sai[CI_R * CI_LD], sbr[CI_R * CI_LD], sbi[CI_R * CI_LD];
  __shared__ double2 sg[64], sA[CI_R];
  constexpr int NTILE = NTL * NTL, TW = (NTILE + 3) / 4;   // tiles, tiles per wave
  const int n = c.n, nn = n * n;
  const int inst = blockIdx.y;
  A += (int64_t)inst * c.dim;
  B += (int64_t)inst * c.dim;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const double* br = same ? sar : sbr;
  const double* bi = same ? sai : sbi;
  dvec4c_t re[TW], im[TW];
#pragma unroll
  for (int j = 0; j < TW; ++j) re[j] = im[j] = dvec4c_t{0.0, 0.0, 0.0, 0.0};
  double2 ga = make_double2(0.0, 0.0);
  for (int base = blockIdx.x * CI_R; base < c.dim; base += gridDim.x * CI_R) {
    __syncthreads();
    ci_fill(c, A, base, sar, sai);
    if (!same) ci_fill(c, B, base, sbr, sbi);
    if (threadIdx.x < CI_R) sA[threadIdx.x] = base + (int)threadIdx.x < c.dim ? A[base + threadIdx.x] : make_double2(0.0, 0.0);
    __syncthreads();
    if (threadIdx.x < (unsigned)nn)
#pragma unroll
      for (int r = 0; r < CI_R; ++r)
        ga = cadd(ga, cjmul(sA[r], make_double2(br[r * CI_LD + threadIdx.x], bi[r * CI_LD + threadIdx.x])));
#pragma unroll
    for (int k0 = 0; k0 < CI_R; k0 += 4) {
      const int kr = (k0 + lk) * CI_LD + li;
#pragma unroll
      for (int j = 0; j < TW; ++j) {
        const int tile = wave + 4 * j < NTILE ? wave + 4 * j : NTILE - 1;
        const int ta = tile / NTL, tb = tile - ta * NTL;
        const double ar = sar[kr + 16 * ta], ai = sai[kr + 16 * ta], xr = br[kr + 16 * tb], xi = bi[kr + 16 * tb];
        re[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, xr, re[j], 0, 0, 0);
        im[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, xi, im[j], 0, 0, 0);
        re[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, xi, re[j], 0, 0, 0);
        im[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, xr, im[j], 0, 0, 0);
      }
    }
  }
  const bool final = gridDim.x == 1;
  double2* pb = part + ((int64_t)inst * gridDim.x + blockIdx.x) * (nn * nn + nn);
  if (threadIdx.x < (unsigned)nn) {
    if (final) {
      sg[threadIdx.x] = ga;
      gamma[(int64_t)inst * nn + threadIdx.x] = ga;
    } else {
      pb[nn * nn + threadIdx.x] = ga;
    }
  }
  if (final) __syncthreads();
  Gamma += (int64_t)inst * nn * nn;
#pragma unroll
  for (int j = 0; j < TW; ++j) {
    const int tile = wave + 4 * j;
    if (tile >= NTILE) continue;
    const int ta = tile / NTL, b = 16 * (tile - ta * NTL) + li;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = 16 * ta + 4 * v + lk;
      if (a >= nn || b >= nn) continue;
      double2 x = make_double2(re[j][v], im[j][v]);
      if (final) {
        const int q = a / n, p = a - q * n, r = b / n, s = b - r * n;
        if (q == r) x = csub(x, sg[p * n + s]);
        Gamma[((p * n + q) * n + r) * n + s] = x;
      } else {
        pb[a * nn + b] = x;
      }
    }
  }
}
// The sums of k_ci_rdm's nblk partial results and the delta term: 16 values per
// workgroup, 16 threads sharing the partials of each.
__global__ void __launch_bounds__(NT) k_ci_rdm_finish(const double2* __restrict__ part, int nblk, int n,
                                                      double2* __restrict__ gamma, double2* __restrict__ Gamma) {
  __shared__ double2 ls[NT / 16][16], lg[NT / 16][16];
  const int nn = n * n, nout = nn * nn + nn;
  const int l = threadIdx.x & 15, w = threadIdx.x >> 4, o = blockIdx.x * 16 + l;
  part += (int64_t)blockIdx.y * nblk * nout;
  gamma += (int64_t)blockIdx.y * nn;
  Gamma += (int64_t)blockIdx.y * nn * nn;
  const bool ok = o < nout, two = ok && o < nn * nn;
  // G[(q, p)][(r, s)] at o; gamma_ps is taken off where q = r
  const int a = two ? o / nn : 0, b = two ? o - a * nn : 0;
  const int q = a / n, p = a - q * n, r = b / n, s = b - r * n;
  const bool dl = two && q == r;
  double2 x = make_double2(0.0, 0.0), y = x;
  if (ok) {
#pragma unroll 4
    for (int k = w; k < nblk; k += NT / 16) {
      x = cadd(x, part[(int64_t)k * nout + o]);
      if (dl) y = cadd(y, part[(int64_t)k * nout + nn * nn + p * n + s]);
    }
  }
  ls[w][l] = x;
  lg[w][l] = y;
  __syncthreads();
  if (w != 0 || !ok) return;
#pragma unroll
  for (int k = 1; k < NT / 16; ++k) {
    x = cadd(x, ls[k][l]);
    y = cadd(y, lg[k][l]);
  }
  if (!two) gamma[o - nn * nn] = x;
  else Gamma[((p * n + q) * n + r) * n + s] = csub(x, y);
}

static void ci_rdms(int ni, const CIDev& c, const double* A, const double* B, double* gamma, double* Gamma,
                    hipStream_t s) {
  const int nn = c.n * c.n, nout = nn * nn + nn;
  const int nblk = c.dim <= 4 * CI_R ? 1 : nblocks(c.dim, CI_R, CI_BLK);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(nblk, ni), dim3(NT), 0, s, c, (const double2*)A, (const double2*)B, A == B ? 1 : 0,
                       (double2*)c.part, (double2*)gamma, (double2*)Gamma);
  };
  if (nn <= 16) go(k_ci_rdm<1>);
  else if (nn <= 32) go(k_ci_rdm<2>);
  else if (nn <= 48) go(k_ci_rdm<3>);
  else go(k_ci_rdm<4>);
  if (nblk > 1)
    hipLaunchKernelGGL(k_ci_rdm_finish, dim3((nout + 15) / 16, ni), dim3(NT), 0, s, (const double2*)c.part, nblk, c.n,
                       (double2*)gamma, (double2*)Gamma);
}
void launch_ci_rdm_full(int ni, const CIDev& c, const double* C, double* gamma, double* Gamma, hipStream_t s) {
  ci_rdms(ni, c, C, C, gamma, Gamma, s);
}
// doubles of CIDev::part per instance
size_t ci_part_doubles(int dim) { return (size_t)nblocks(dim, CI_R, CI_BLK) * 2 * (4096 + 64); }

// h'_pq = h_pq - 1/2 sum_q' g_pq'q'q
__global__ void k_ci_hprime(const double2* __restrict__ h, const double2* __restrict__ g, int n,
                            double2* __restrict__ hp) {
  const int nn = n * n;
  h += (int64_t)blockIdx.x * nn;
  g += (int64_t)blockIdx.x * nn * nn;
  hp += (int64_t)blockIdx.x * nn;
  for (int o = threadIdx.x; o < nn; o += blockDim.x) {
    int p = o / n, q = o % n;
    double2 s = h[o];
    for (int k = 0; k < n; ++k) s = csub(s, cscale(0.5, g[((p * n + k) * n + k) * n + q]));
    hp[o] = s;
  }
}
void launch_ci_hprime(int ni, const CIDev& c, const double* h, const double* g, hipStream_t s) {
  hipLaunchKernelGGL(k_ci_hprime, dim3(ni), dim3(64), 0, s, (const double2*)h, (const double2*)g, c.n,
                     (double2*)c.hp);
}

// T[J][pq] = h'_pq C[J] + 1/2 sum_rs g_pqrs (E_rs C)(J): a workgroup takes 16
// determinants, their excited amplitudes in LDS and wave w the pairs pq of tile
// w, whose rows of g it holds in registers; FP64 matrix-core tiles (lane layout
// of k_moments_mfma).
template <int NTL>
__global__ void __launch_bounds__(NT) k_ci_T(CIDev c, const double2* __restrict__ C, const double2* __restrict__ g) {
  typedef double dvec4c_t __attribute__((ext_vector_type(4)));
  __shared__ double sr[16 * CI_LD], si[16 * CI_LD];
  const int nn = c.n * c.n, inst = blockIdx.y;
  C += (int64_t)inst * c.dim;
  g += (int64_t)inst * nn * nn;
  const double2* hp = (const double2*)c.hp + (int64_t)inst * nn;
  double2* T = (double2*)c.T + (int64_t)inst * c.dim * nn;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int base = blockIdx.x * 16, pq = 16 * wave + li;
  double2 gv[4 * NTL];   // g[pq][4 k + lk]
#pragma unroll
  for (int k = 0; k < 4 * NTL; ++k) {
    const int rs = 4 * k + lk;
    gv[k] = (pq < nn && rs < nn) ? ldg2(g, (int64_t)pq * nn + rs) : make_double2(0.0, 0.0);
  }
  ci_fill(c, C, base, sr, si);
  __syncthreads();
  dvec4c_t re = dvec4c_t{0.0, 0.0, 0.0, 0.0}, im = re;
#pragma unroll
  for (int k = 0; k < 4 * NTL; ++k) {
    const double ar = sr[li * CI_LD + 4 * k + lk], ai = si[li * CI_LD + 4 * k + lk];
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, gv[k].x, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, gv[k].y, im, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, gv[k].y, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, gv[k].x, im, 0, 0, 0);
  }
  if (pq >= nn) return;
  const double2 h = hp[pq];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int J = base + 4 * v + lk;
    if (J < c.dim) T[(int64_t)J * nn + pq] = cadd(cmul(h, C[J]), make_double2(0.5 * re[v], 0.5 * im[v]));
  }
}

// sigma[J] = sum_pq (E_pq T_pq)(J), G lanes (a power of two) per determinant
// sharing its pairs.
template <int G>
__global__ void __launch_bounds__(NT) k_ci_sigma(CIDev c, double2* __restrict__ sigma) {
  const int nn = c.n * c.n, inst = blockIdx.y;
  const double2* T = (const double2*)c.T + (int64_t)inst * c.dim * nn;
  sigma += (int64_t)inst * c.dim;
  const int J = (blockIdx.x * NT + threadIdx.x) / G, l = threadIdx.x & (G - 1);
  double2 s = make_double2(0.0, 0.0);
  if (J < c.dim) {
    const int Ja = J / c.NB, Jb = J - Ja * c.NB;
    for (int pq = l; pq < nn; pq += G) {
      const int ta = gbl(c.exa)[Ja * nn + pq], tb = gbl(c.exb)[Jb * nn + pq];
      if (ta >= 0) s = cadd(s, cscale((ta >> 30) ? -1.0 : 1.0, ldg2(T, (int64_t)((ta & 0x3fffffff) * c.NB + Jb) * nn + pq)));
      if (tb >= 0) s = cadd(s, cscale((tb >> 30) ? -1.0 : 1.0, ldg2(T, (int64_t)(Ja * c.NB + (tb & 0x3fffffff)) * nn + pq)));
    }
  }
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) {
    s.x += __shfl_xor(s.x, o, G);
    s.y += __shfl_xor(s.y, o, G);
  }
  if (J < c.dim && l == 0) sigma[J] = s;
}

static void launch_ci_sigma(int ni, const CIDev& c, const double* C, const double* g, double* sigma, hipStream_t s) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((c.dim + 15) / 16, ni), dim3(NT), 0, s, c, (const double2*)C, (const double2*)g);
  };
  if (c.n <= 4) go(k_ci_T<1>);
  else if (c.n <= 5) go(k_ci_T<2>);
  else if (c.n <= 6) go(k_ci_T<3>);
  else go(k_ci_T<4>);
  if (c.n <= 2)
    hipLaunchKernelGGL(k_ci_sigma<4>, dim3(nblocks((int64_t)c.dim * 4), ni), dim3(NT), 0, s, c, (double2*)sigma);
  else if (c.n <= 4)
    hipLaunchKernelGGL(k_ci_sigma<16>, dim3(nblocks((int64_t)c.dim * 16), ni), dim3(NT), 0, s, c, (double2*)sigma);
  else
    hipLaunchKernelGGL(k_ci_sigma<64>, dim3(nblocks((int64_t)c.dim * 64), ni), dim3(NT), 0, s, c, (double2*)sigma);
}

void launch_ci_trdm(int ni, const CIDev& c, const double* A, const double* Bv, double* gamma, double* Gamma,
                    hipStream_t s) {
  ci_rdms(ni, c, A, Bv, gamma, Gamma, s);
}

// sigma = (sum h_pq E_pq + 1/2 sum g_pqrs (E_pq E_rs - delta_qr E_ps)) C for
// general h and g; overwrites the shared h' of the CI space.
void launch_ci_apply(int ni, const CIDev& c, const double* h, const double* g, const double* C, double* sigma,
                     hipStream_t s) {
  launch_ci_hprime(ni, c, h, g, s);
  launch_ci_sigma(ni, c, C, g, sigma, s);
}

// One Lanczos/Arnoldi step on the CI space inside one workgroup: w is
// orthogonalised twice against Q_0..Q_k (full re-orthogonalisation, the dots of
// a pass together), H column k filled, h_{k+1,k} = |w| (breakdown: scale 0,
// m_eff = k+1), Q_{k+1} = w / h.  At most CI_M = 12 vectors.
constexpr int CI_M = 12;
__global__ void __launch_bounds__(1024) k_ci_lanczos_step(int dim, double2* const* __restrict__ Q, int k,
                                                          double2* __restrict__ w, double2* __restrict__ H, int m_max,
                                                          double* __restrict__ scal, int last) {
  constexpr int NV = 2 * CI_M;
  __shared__ double lw[16][NV];
  __shared__ double hs[NV];
  const int inst = blockIdx.x, wid = threadIdx.x >> 6;
  const int64_t vo = (int64_t)inst * dim;
  w += vo;
  H += (int64_t)inst * (m_max + 1) * m_max + (int64_t)(m_max + 1) * k;
  scal += 8 * inst;
  double nrm = 0.0;
  for (int pass = 0; pass < 2; ++pass) {
    double acc[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) acc[j] = 0.0;
    for (int i = threadIdx.x; i < dim; i += 1024) {
      const double2 x = ldg2(w, i);
#pragma unroll
      for (int j = 0; j < CI_M; ++j)
        if (j <= k) {
          const double2 q = ldg2(Q[j], vo + i);
          acc[2 * j] += q.x * x.x + q.y * x.y;
          acc[2 * j + 1] += q.x * x.y - q.y * x.x;
        }
    }
    wave_sum_values(acc, lw[wid]);
    __syncthreads();
    if (threadIdx.x < (unsigned)(2 * (k + 1))) {
      double t = 0.0;
#pragma unroll
      for (int v = 0; v < 16; ++v) t += lw[v][threadIdx.x];
      hs[threadIdx.x] = t;
      double* hp = (double*)H + threadIdx.x;
      if (pass == 0) *hp = t;
      else *hp += t;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < dim; i += 1024) {
      double2 x = ldg2(w, i);
#pragma unroll
      for (int j = 0; j < CI_M; ++j)
        if (j <= k) x = csub(x, cmul(make_double2(hs[2 * j], hs[2 * j + 1]), ldg2(Q[j], vo + i)));
      w[i] = x;
      if (pass == 1) nrm += x.x * x.x + x.y * x.y;
    }
  }
  if (last) return;
  nrm = wave_sum(nrm);
  if ((threadIdx.x & 63) == 0) lw[wid][0] = nrm;
  __syncthreads();
  nrm = 0.0;
#pragma unroll
  for (int v = 0; v < 16; ++v) nrm += lw[v][0];
  nrm = sqrt(nrm);
  const double2 dd = H[k];
  const bool brk = !(nrm > 1e-14 * fmax(1.0, hypot(dd.x, dd.y)));
  const double sc = brk ? 0.0 : 1.0 / nrm;
  if (threadIdx.x == 0) {
    H[k + 1] = make_double2(brk ? 0.0 : nrm, 0.0);
    if (brk && scal[4] > k + 1) scal[4] = k + 1;
  }
  for (int i = threadIdx.x; i < dim; i += 1024) Q[k + 1][vo + i] = cscale(sc, ldg2(w, i));
}

// The whole CI exponential of a small space (dim <= CI_SD determinants, dim n^2
// <= CI_ST) in one workgroup per instance: vectors, amplitudes and the
// Hessenberg matrix stay in LDS, so a step is a few barriers instead of four
// launches.  Same process as the launches above.  Measured: 4 determinants, 22 us against
// about 160 us in 19 launches; 9 determinants, 59 against 440 us
constexpr int CI_SD = 64, CI_ST = 1024;
struct CiSmallLds {
  double2 Q[CI_M][CI_SD], w[CI_SD], D[CI_ST], T[CI_ST], H[(CI_M + 1) * CI_M], hs[CI_M];
  double nrm;
};
__global__ void __launch_bounds__(NT) k_ci_small(CIDev c, const double2* __restrict__ g, int m,
                                                 double2* __restrict__ Cv, double tau_re, double tau_im,
                                                 int normalize) {
  __shared__ CiSmallLds L;
  __shared__ ExpmLds<CI_M> X;
  const int nn = c.n * c.n, dim = c.dim, inst = blockIdx.x, lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  g += (int64_t)inst * nn * nn;
  Cv += (int64_t)inst * dim;
  const double2* hp = (const double2*)c.hp + (int64_t)inst * nn;
  // |v|, v in LDS with at most 64 entries (the first wave; every thread gets it)
  auto norm_of = [&](const double2* v) {
    if (wid == 0) {
      double t = lane < dim ? v[lane].x * v[lane].x + v[lane].y * v[lane].y : 0.0;
      t = wave_sum(t);
      if (lane == 0) L.nrm = sqrt(t);
    }
    __syncthreads();
    return L.nrm;
  };
  if ((int)threadIdx.x < dim) L.w[threadIdx.x] = Cv[threadIdx.x];
  for (int e = threadIdx.x; e < (CI_M + 1) * CI_M; e += NT) L.H[e] = make_double2(0.0, 0.0);
  __syncthreads();
  const double beta = norm_of(L.w);
  if ((int)threadIdx.x < dim) L.Q[0][threadIdx.x] = cscale(beta > 0.0 ? 1.0 / beta : 0.0, L.w[threadIdx.x]);
  int m_eff = m;
  for (int k = 0; k < m; ++k) {
    __syncthreads();
    const double2* C = L.Q[k];
    for (int e = threadIdx.x; e < dim * nn; e += NT) L.D[e] = ci_excited(c, C, e / nn, e % nn);
    __syncthreads();
    for (int e = threadIdx.x; e < dim * nn; e += NT) {
      const int J = e / nn, pq = e - J * nn;
      double2 t = make_double2(0.0, 0.0);
      for (int rs = 0; rs < nn; ++rs) t = cadd(t, cmul(ldg2(g, pq * nn + rs), L.D[J * nn + rs]));
      L.T[e] = cadd(cmul(hp[pq], C[J]), cscale(0.5, t));
    }
    __syncthreads();
    for (int J = wid; J < dim; J += NT / 64) {   // a wave per determinant
      const int Ja = J / c.NB, Jb = J - Ja * c.NB;
      double2 s = make_double2(0.0, 0.0);
      if (lane < nn) {
        const int ta = gbl(c.exa)[Ja * nn + lane], tb = gbl(c.exb)[Jb * nn + lane];
        if (ta >= 0) s = cscale((ta >> 30) ? -1.0 : 1.0, L.T[((ta & 0x3fffffff) * c.NB + Jb) * nn + lane]);
        if (tb >= 0) s = cadd(s, cscale((tb >> 30) ? -1.0 : 1.0, L.T[(Ja * c.NB + (tb & 0x3fffffff)) * nn + lane]));
      }
      s.x = wave_sum(s.x);
      s.y = wave_sum(s.y);
      if (lane == 0) L.w[J] = s;
    }
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
      for (int j = wid; j <= k; j += NT / 64) {
        double2 t = lane < dim ? cjmul(L.Q[j][lane], L.w[lane]) : make_double2(0.0, 0.0);
        t.x = wave_sum(t.x);
        t.y = wave_sum(t.y);
        if (lane == 0) {
          L.hs[j] = t;
          L.H[j + (CI_M + 1) * k] = pass == 0 ? t : cadd(L.H[j + (CI_M + 1) * k], t);
        }
      }
      __syncthreads();
      if ((int)threadIdx.x < dim) {
        double2 x = L.w[threadIdx.x];
        for (int j = 0; j <= k; ++j) x = csub(x, cmul(L.hs[j], L.Q[j][threadIdx.x]));
        L.w[threadIdx.x] = x;
      }
      __syncthreads();
    }
    if (k == m - 1) break;
    const double nrm = norm_of(L.w);
    const double2 dd = L.H[k + (CI_M + 1) * k];
    if (!(nrm > 1e-14 * fmax(1.0, hypot(dd.x, dd.y)))) {   // breakdown: the space ends here
      m_eff = k + 1;
      break;
    }
    if (threadIdx.x == 0) L.H[(k + 1) + (CI_M + 1) * k] = make_double2(nrm, 0.0);
    if ((int)threadIdx.x < dim) L.Q[k + 1][threadIdx.x] = cscale(1.0 / nrm, L.w[threadIdx.x]);
  }
  __syncthreads();
  const double2 f = make_double2(tau_im, -tau_re);
  for (int e = threadIdx.x; e < m_eff * m_eff; e += NT) {
    const int i = e / m_eff, j = e - i * m_eff;
    X.A[e] = cmul(f, L.H[i + (CI_M + 1) * j]);
  }
  expm_lds(X, m_eff);
  if ((int)threadIdx.x < dim) {
    double2 s = make_double2(0.0, 0.0);
    for (int j = 0; j < m_eff; ++j) s = cadd(s, cmul(cscale(beta, X.T[j * m_eff]), L.Q[j][threadIdx.x]));
    L.w[threadIdx.x] = s;
  }
  __syncthreads();
  const double fn = normalize ? 1.0 / norm_of(L.w) : 1.0;
  if ((int)threadIdx.x < dim) Cv[threadIdx.x] = cscale(fn, L.w[threadIdx.x]);
}

__global__ void __launch_bounds__(1024) k_ci_start(int dim, const double2* __restrict__ C, double2* __restrict__ Q0,
                                                   double* __restrict__ scal, int m, double2* __restrict__ H,
                                                   int m_max) {
  __shared__ double red[32];
  const int inst = blockIdx.x;
  C += (int64_t)inst * dim;
  Q0 += (int64_t)inst * dim;
  H += (int64_t)inst * (m_max + 1) * m_max;
  scal += 8 * inst;
  double s = 0.0;
  for (int i = threadIdx.x; i < dim; i += blockDim.x) s += C[i].x * C[i].x + C[i].y * C[i].y;
  s = wave_sum(s);
  int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) red[wid] = s;
  __syncthreads();
  double t = 0.0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
  double beta = sqrt(t);
  const double ib = beta > 0.0 ? 1.0 / beta : 0.0;  // a zero vector stays zero
  for (int i = threadIdx.x; i < dim; i += blockDim.x) Q0[i] = cscale(ib, C[i]);
  for (int i = threadIdx.x; i < (m_max + 1) * m_max; i += blockDim.x) H[i] = make_double2(0.0, 0.0);
  if (threadIdx.x == 0) {
    scal[0] = beta;
    scal[4] = m;
    scal[3] = 0.0;
  }
}

__global__ void __launch_bounds__(1024) k_ci_combine(int dim, double2* const* __restrict__ Q, int m, int m_max,
                                                     const double2* __restrict__ y, double2* __restrict__ C,
                                                     int normalize) {
  __shared__ double red[32];
  const int inst = blockIdx.x;
  const int64_t vo = (int64_t)inst * dim;
  y += (int64_t)inst * m_max;
  C += vo;
  double s2 = 0.0;
  for (int i = threadIdx.x; i < dim; i += blockDim.x) {
    double2 s = make_double2(0.0, 0.0);
    for (int j = 0; j < m; ++j) s = cadd(s, cmul(y[j], Q[j][vo + i]));
    C[i] = s;
    s2 += s.x * s.x + s.y * s.y;
  }
  if (!normalize) return;
  s2 = wave_sum(s2);
  int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) red[wid] = s2;
  __syncthreads();
  double t = 0.0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
  double f = 1.0 / sqrt(t);
  for (int i = threadIdx.x; i < dim; i += blockDim.x) C[i] = cscale(f, C[i]);
}

void launch_ci_lanczos(int ni, const CIDev& c, double* const* Qdev, double* const* Qhost, int m, const double* g,
                       double* Cvec, Krylov& K, double tau_re, double tau_im, int normalize, hipStream_t s) {
  if (c.dim <= CI_SD && c.dim * c.n * c.n <= CI_ST && m <= CI_M) {
    hipLaunchKernelGGL(k_ci_small, dim3(ni), dim3(NT), 0, s, c, (const double2*)g, m, (double2*)Cvec, tau_re, tau_im,
                       normalize);
    return;
  }
  hipLaunchKernelGGL(k_ci_start, dim3(ni), dim3(1024), 0, s, c.dim, (const double2*)Cvec, (double2*)Qhost[0], K.scal,
                     m, (double2*)K.H, K.m_max);
  for (int k = 0; k < m; ++k) {
    launch_ci_sigma(ni, c, Qhost[k], g, c.w, s);
    hipLaunchKernelGGL(k_ci_lanczos_step, dim3(ni), dim3(1024), 0, s, c.dim, (double2* const*)Qdev, k, (double2*)c.w,
                       (double2*)K.H, K.m_max, K.scal, (k == m - 1) ? 1 : 0);
  }
  hipLaunchKernelGGL(k_expm, dim3(1, ni), dim3(NT), 0, s, (const double2*)K.H, K.m_max, tau_re, tau_im, K.scal,
                     (double2*)K.y, 0, 0.0);
  hipLaunchKernelGGL(k_ci_combine, dim3(ni), dim3(1024), 0, s, c.dim, (double2* const*)Qdev, m, K.m_max,
                     (const double2*)K.y, (double2*)Cvec, normalize);
}

}  // namespace mh
