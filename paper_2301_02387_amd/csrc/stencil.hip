// Node-centric, atomic-free application of the one-body and Poisson
// operators (Sec. III.A tensor-product Lagrange basis on Gauss-Lobatto
// points; Eq. discretized_eom), and the Jacobi-preconditioned CG on the
// assembled Poisson operator.
//
// The element stiffness (h/2)(A x W x W + W x A x W + W x W x A) couples a
// node only to the nodes on its three coordinate lines inside each cell
// holding it (W is diagonal).  Each node therefore gathers its assembled
// value directly, from the row of coupled nodes laid out when the operator is
// created.  The result is written once, with no scatter and no atomics.  Node-diagonal
// terms (nuclear potential, field, mean field) are added by the same
// thread; for DoFs that are not hanging-node masters the mass solve and
// the projector term are applied in the same pass, so the output is final.
// Masters and hanging nodes hand their load values to a small gather
// kernel (the transposed constraints C^T) and the interface mass solve.
//
// Lane layout: L lanes per node (L a power of two >= the number of
// columns); lane = orbital (complex) or Poisson column (real).  Nodes are
// numbered in first-touch order over Morton-sorted cells, so the lines a
// wave reads are mostly shared with its neighbours and hit in L1/L2.
// Batched launches: instance blockIdx.y (kernels.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "devutil.hpp"
#include "kernels.hpp"
#include "mg.hpp"

namespace mh {

#define INSTANCE const DevMesh& d = dm[blockIdx.y]

// --------------------------------------------------------------------------
// Rows of the one-body operator.  Entry e = (cell t, direction, line point q)
// of node i couples it to one node of a line through it; the row holds each
// coupled node once, in order of first appearance (at most 8 cells x 3 lines x
// (P - 1) + 1).  Stiffness (1/2) K; S along the field direction e: per cell
// (h/2)^2 (Qs x W x W) along x and likewise along y and z.  Complex scaling: a
// cell's stiffness and derivative loads along d take the contour factors
// e^{i (s - 2 b_d) theta} and e^{i (s - b_d) theta} (s scaled directions, b_d
// whether d is one), the node's sum rho = m / m_theta.
// --------------------------------------------------------------------------
template <int P>
__device__ __forceinline__ int orb_entry_col(const DevMesh& d, int64_t i, int e) {
  const int q = e % P, dir = (e / P) % 3, t = e / (3 * P);
  const int code = gbl(d.node_inc)[i * 8 + t];
  if (code < 0) return -1;
  const int loc = code & 63, a = loc % P, b = (loc / P) % P, c = loc / (P * P);
  const int l = dir == 0 ? (c * P + b) * P + q : dir == 1 ? (c * P + q) * P + a : (q * P + b) * P + a;
  const int j = gbl(d.cell_nodes)[(int64_t)(code >> 6) * (P * P * P) + l];
  return j < d.NE ? j : -1;
}
template <int P>
__device__ __forceinline__ void orb_entry_add(const DevMesh& d, int64_t i, int e, double& k, double& sv, double2& kc,
                                              double2& sc) {
  const int q = e % P, dir = (e / P) % 3, t = e / (3 * P);
  const int code = gbl(d.node_inc)[i * 8 + t], loc = code & 63;
  const int64_t K = code >> 6;
  const int x[3] = {loc % P, (loc / P) % P, loc / (P * P)};
  const int a = x[dir], o1 = x[dir == 0 ? 1 : 0], o2 = x[dir == 2 ? 1 : 2];
  const double h2 = gbl(d.cell_hh)[K], ww = d.w[o1] * d.w[o2];
  const double fk = 0.5 * h2 * ww * d.A[a * P + q], fs = h2 * h2 * d.pol[dir] * ww * d.Qs[a * P + q];
  k += fk;
  sv += fs;
  if (d.ecs) {
    const int bits = gbl(d.ecs_code)[K], bd = (bits >> dir) & 1;
    const int s = (bits & 1) + ((bits >> 1) & 1) + ((bits >> 2) & 1);
    auto pw = [&](int z) { return make_double2(d.ecs_pw[2 * (z + 2)], d.ecs_pw[2 * (z + 2) + 1]); };
    kc = cadd(kc, cscale(fk, pw(s - 2 * bd)));
    sc = cadd(sc, cscale(fs, pw(s - bd)));
  }
}
template <int P, bool FILL>
__global__ void __launch_bounds__(NT) k_orb_row_build(const DevMesh* __restrict__ dm) {
  INSTANCE;
  int32_t* col = const_cast<int32_t*>(d.or_col);
  double* k = const_cast<double*>(d.or_k);
  double* sv = const_cast<double*>(d.or_s);
  double2 *kc = (double2*)const_cast<double*>(d.or_kc), *sc = (double2*)const_cast<double*>(d.or_sc);
  constexpr int E = 24 * P;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < d.NE; i += (int64_t)gridDim.x * NT) {
    int cols[E], m = 0;
    for (int e = 0; e < E; ++e) cols[e] = orb_entry_col<P>(d, i, e);
    const int64_t at = FILL ? gbl(d.or_ptr)[i] : 0;
    for (int e = 0; e < E; ++e) {
      const int j = cols[e];
      if (j < 0) continue;
      if (FILL) {
        double kv = 0.0, s = 0.0;
        double2 kz = make_double2(0.0, 0.0), sz = kz;
        for (int f = e; f < E; ++f)
          if (cols[f] == j) {
            orb_entry_add<P>(d, i, f, kv, s, kz, sz);
            cols[f] = -1;
          }
        col[at + m] = j;
        k[at + m] = kv;
        sv[at + m] = s;
        if (d.ecs) {
          const double2 rho = make_double2(d.ecs_rho[2 * i], d.ecs_rho[2 * i + 1]);
          kc[at + m] = cmul(rho, kz);
          sc[at + m] = cmul(rho, sz);
        }
      } else {
        for (int f = e; f < E; ++f)
          if (cols[f] == j) cols[f] = -1;
      }
      ++m;
    }
    if (!FILL) const_cast<int32_t*>(d.or_ptr)[i + 1] = m;
  }
}
template <bool FILL>
static void orb_row_build(const Batch& b, hipStream_t s) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(nblocks(b.mx.NE, NT, 4096), b.ni), dim3(NT), 0, s, b.dm);
  };
  if (b.mx.P == 2) go(k_orb_row_build<2, FILL>);
  else if (b.mx.P == 3) go(k_orb_row_build<3, FILL>);
  else go(k_orb_row_build<4, FILL>);
}
void launch_orb_row_count(const Batch& b, hipStream_t s) { orb_row_build<false>(b, s); }
void launch_orb_row_fill(const Batch& b, hipStream_t s) { orb_row_build<true>(b, s); }

// --------------------------------------------------------------------------
// Orbital operator.  mode 0: F = load vector; 1: M^-1 F; 2: M^-1 F - v lam.
// diag_mode 0: one-body stiffness; 1: with the potential and the field; 2: with
// the mean field; 3: dipole weights only; 4: momentum along the field.
// Non-master DoFs get their final value in `out`; masters and hanging nodes
// store the load value in `acc`.
//
// One pass over the rows above: L lanes (n rounded up to a power of two) hold
// the node's orbitals, GR groups of them share its entries.  What the node adds
// itself (diagonal weights, its n^2 mean-field values) is requested before the
// row is gathered.  OP_K: stiffness; OP_S: the first-derivative term -i a.S u of
// the velocity gauge (a = A(t) e, or e alone for the momentum); CX: instances
// with complex scaling take the complex rows (their potential and field weights
// are the continued ones, in units of the real mass; the mean-field load is
// unchanged).
// Bound by the gathers out of L2 (13 rows a node at Q3) and, at eight orbitals,
// by HBM (512 B of mean-field values a node beside 128 B read and written);
// where few nodes are, by the chain row -> index -> gather.  Before, the line
// sums ran cell by cell (indices of every line of up to eight cells), or the
// assembled Poisson operator on 2n real columns and a second pass over the nodes.
// Measured, before -> rows: H2O (1.65 M nodes x 8 orbitals) 353 + 462 -> 539 us,
// its momentum 1650 -> 359; on the Q1 mesh, velocity gauge with complex scaling
// (234,000 x 8) 274 -> 113; 16 H2 (75,900 x 2 each) 144 + 52 -> 148; H2 14.0 +
// 6.6 -> 12.9; 3 orbitals in the velocity gauge (Q2) 27 -> 10.4 us.
// --------------------------------------------------------------------------
template <int L, int GR, bool OP_K, bool OP_S, bool CX, bool MF>
__global__ void __launch_bounds__(NT, OP_S && MF ? 3 : 4) k_orb_rows(const DevMesh* __restrict__ dm,
                                                             const double2* __restrict__ u,
                                                             const double* __restrict__ Ef, int diag_mode,
                                                             const double* __restrict__ Upk,
                                                             const double2* __restrict__ ginv, int mode,
                                                             const double2* __restrict__ lam,
                                                             double2* __restrict__ out, double2* __restrict__ acc) {
  INSTANCE;
  constexpr int LR = L * GR, RW = 64 / LR, U = GR > 2 ? 16 / GR : CX ? 4 : 8, NQ = (L + GR - 1) / GR, LS = L + 1;
  // per wave: the rows' packed mean-field matrices (row stride L + 1: lanes p and
  // rows fall on different banks), orbitals and mean-field products
  __shared__ double sU[MF ? NT / 64 : 1][MF ? RW * L * LS : 1];
  __shared__ double2 su[NT / 64][RW * L], sz[NT / 64][MF ? RW * L : 1];
  __shared__ double2 sg[MF ? L * L : 1], sl[L * L];   // S^-1 transposed, lambda: row q, lane p
  const int n = d.n;
  const int64_t o = d.oE * n;
  u += o;
  out += o;
  acc += o;
  Upk += d.oE * n * n;
  const int lane = (int)(threadIdx.x % LR), p = lane % L, grp = lane / L;
  const int wave = (int)(threadIdx.x >> 6), slot = (int)(threadIdx.x & 63) / LR;
  const bool act = p < n && grp == 0;
  const int pc = min(p, n - 1);   // lanes past the last orbital repeat it and write nothing
  for (int f = threadIdx.x; f < n * n; f += NT) {
    const int r = f / n, c = f - r * n;
    if (MF) sg[c * L + r] = ldg2(ginv, (int64_t)blockIdx.y * n * n + f);
    if (mode == 2) sl[r * L + c] = ldg2(lam, (int64_t)blockIdx.y * n * n + f);
  }
  if (MF || mode == 2) __syncthreads();
  const double E = (diag_mode == 1 || diag_mode == 2) ? Ef[0] * d.E0 : 0.0;
  const double av = diag_mode == 4 ? 1.0 : E;
  const double Elen = d.gauge == 1 ? 0.0 : E;   // the length-gauge term only in the length gauge
  const bool cx = CX && d.ecs;
  const bool diag = diag_mode >= 1 && diag_mode <= 3;
  double* Up = &sU[MF ? wave : 0][MF ? slot * L * LS : 0];
  double2* Us = &su[wave][slot * L];
  double2* Zs = &sz[wave][MF ? slot * L : 0];
  const auto* colp = gbl(d.or_col);
  const auto* kp = gbl(d.or_k);
  const auto* sp = gbl(d.or_s);
  const XcdSweep sw = xcd_sweep(d.NE, NT / LR, d.sched_orb & 1);
  // all LR lanes of a node share i, so a node group enters and leaves together
  for (int i = (int)sw.start + (int)threadIdx.x / LR; i < (int)sw.end; i += (int)sw.step) {
    const int64_t at = (int64_t)i * n + pc;
    int beg = 0, end = 0, jn[U];
    if (OP_K || OP_S) {
      beg = gbl(d.or_ptr)[i] + grp;
      end = gbl(d.or_ptr)[i + 1];
#pragma unroll
      for (int h = 0; h < U; ++h) jn[h] = colp[min(beg + h * GR, end - 1)];   // a row holds its own node at least
    }
    const double2 ui = ldg2(u, at);
    double2 dg = make_double2(0.0, 0.0);
    if (diag) {
      if (cx && diag_mode != 3) {
        const double2 vc = ldg2(d.ecs_v, i), zc = ldg2(d.ecs_mz, i);
        dg = make_double2(vc.x + Elen * zc.x, vc.y + Elen * zc.y);
      } else {
        dg.x = diag_mode == 3 ? gbl(d.mz)[i] : gbl(d.v)[i] + Elen * gbl(d.mz)[i];
      }
    }
    double up[NQ], mass = 0.0;
    if (MF) {
#pragma unroll
      for (int h = 0; h < NQ; ++h) up[h] = gbl(Upk)[(int64_t)i * (n * n) + min(h * GR + grp, n - 1) * n + pc];
      mass = gbl(d.m)[i];
    }
    const bool dof = i < d.N;
    const int mi = dof ? gbl(d.ma_index)[i] : -1;
    const double im = dof && mi < 0 && mode != 0 ? gbl(d.inv_mass)[i] : 0.0;
    // the row: y = sum k u, t = sum s u; the next round's nodes are requested
    // before this round's gathers, entries past the end count zero
    double2 y = make_double2(0.0, 0.0), t = y;
    if (OP_K || OP_S) {
      for (int e0 = beg; e0 - grp < end; e0 += U * GR) {
        double2 k[U], sv[U], v[U];
#pragma unroll
        for (int h = 0; h < U; ++h) v[h] = ldg2(u, (int64_t)((unsigned)jn[h] * (unsigned)n + (unsigned)pc));
#pragma unroll
        for (int h = 0; h < U; ++h) {
          const int e = e0 + h * GR, ec = min(e, end - 1);
          const bool in = e < end;
          if (OP_K) {
            if (cx) k[h] = ldg2(d.or_kc, ec);
            else k[h] = make_double2(kp[ec], 0.0);
            k[h].x = in ? k[h].x : 0.0;
            if (CX) k[h].y = in ? k[h].y : 0.0;
          }
          if (OP_S) {
            if (cx) sv[h] = ldg2(d.or_sc, ec);
            else sv[h] = make_double2(sp[ec], 0.0);
            sv[h].x = in ? sv[h].x : 0.0;
            if (CX) sv[h].y = in ? sv[h].y : 0.0;
          }
        }
        if (e0 - grp + U * GR < end) {
#pragma unroll
          for (int h = 0; h < U; ++h) jn[h] = colp[min(e0 + (U + h) * GR, end - 1)];
        }
#pragma unroll
        for (int h = 0; h < U; ++h) {
          if (CX) {
            if (OP_K) y = cadd(y, cmul(k[h], v[h]));
            if (OP_S) t = cadd(t, cmul(sv[h], v[h]));
          } else {
            if (OP_K) y = cadd(y, cscale(k[h].x, v[h]));
            if (OP_S) t = cadd(t, cscale(sv[h].x, v[h]));
          }
        }
      }
    }
    if (OP_S) {  // -i a t
      y.x += av * t.y;
      y.y -= av * t.x;
    }
    // The groups split the sums over orbitals too: z_p = sum_q U_pq u_q (U
    // Hermitian, packed: Up[o][q] = Re U_oq, Up[q][o] = Im U_oq for o < q),
    // S^-1 z and u lambda.
    double2 lm = make_double2(0.0, 0.0);
    if (MF || mode == 2) {
      if (grp == 0) Us[p] = ui;
      if (MF) {
#pragma unroll
        for (int h = 0; h < NQ; ++h)
          if (h * GR + grp < L) Up[(h * GR + grp) * LS + p] = up[h];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      double2 z = make_double2(0.0, 0.0);
#pragma unroll
      for (int h = 0; h < NQ; ++h) {
        const int q = h * GR + grp;
        if (q < n) {
          const double2 uq = Us[q];
          if (MF) {
            const double a = Up[p * LS + q], c = Up[q * LS + p];
            z = cadd(z, cmul(make_double2(p <= q ? a : c, p < q ? c : (p > q ? -a : 0.0)), uq));
          }
          if (mode == 2) lm = cadd(lm, cmul(sl[q * L + p], uq));
        }
      }
      if (MF) {
#pragma unroll
        for (int off = LR / 2; off >= L; off >>= 1) {
          z.x += __shfl_xor(z.x, off, 64);
          z.y += __shfl_xor(z.y, off, 64);
        }
        if (grp == 0) Zs[p] = z;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        double2 wv = make_double2(0.0, 0.0);
#pragma unroll
        for (int h = 0; h < NQ; ++h) {
          const int q = h * GR + grp;
          if (q < n) wv = cadd(wv, cmul(sg[q * L + p], Zs[q]));
        }
        y.x += mass * wv.x;
        y.y += mass * wv.y;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();  // the slices are rewritten for the wave's next nodes
    }
    if (diag && grp == 0) y = cadd(y, cmul(dg, ui));
    y = make_double2(im != 0.0 ? im * y.x - lm.x : y.x, im != 0.0 ? im * y.y - lm.y : y.y);
#pragma unroll
    for (int off = LR / 2; off >= L; off >>= 1) {
      y.x += __shfl_xor(y.x, off, 64);
      y.y += __shfl_xor(y.y, off, 64);
    }
    if (!act) continue;
    if (dof && mi < 0) out[at] = y;
    else acc[at] = y;
  }
}

template <int L, int GR>
static void launch_orb_rows(const Batch& b, const double* u, const double* Ef, int diag_mode, const double* Upk,
                            const double* ginv, int mode, const double* lam, double* out, double* acc, hipStream_t s) {
  const bool vel = b.mx.gauge == 1 && (diag_mode == 1 || diag_mode == 2), cx = b.mx.ecs && diag_mode <= 2;
  const bool mf = diag_mode == 2;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(xcd_grid(b.mx.NE, NT / (L * GR), b.mx.grid_orb), b.ni), dim3(NT), 0, s, b.dm,
                       (const double2*)u, Ef, diag_mode, Upk, (const double2*)ginv, mode, (const double2*)lam,
                       (double2*)out, (double2*)acc);
  };
  if (diag_mode == 3) go(k_orb_rows<L, GR, false, false, false, false>);
  else if (diag_mode == 4) go(k_orb_rows<L, GR, false, true, false, false>);
  else if (vel && cx) mf ? go(k_orb_rows<L, GR, true, true, true, true>) : go(k_orb_rows<L, GR, true, true, true, false>);
  else if (vel) mf ? go(k_orb_rows<L, GR, true, true, false, true>) : go(k_orb_rows<L, GR, true, true, false, false>);
  else if (cx) mf ? go(k_orb_rows<L, GR, true, false, true, true>) : go(k_orb_rows<L, GR, true, false, true, false>);
  else mf ? go(k_orb_rows<L, GR, true, false, false, true>) : go(k_orb_rows<L, GR, true, false, false, false>);
}

// Lane groups per node: four (of one orbital eight) while the lanes of a single
// group leave the chip idle, below 2^17 (one orbital 2^14, two 2^18), since a
// node's entries are then a chain; above that one, with one and two orbitals as many
// as read a node's entries in whole sectors.  Measured with 1, 2, 4, 8 groups, us:
// 8 orbitals  4,583 nodes 9.3, 6.4, 5.9, 6.4;  12,468 10.1, 9.3, 9.4, 10.9;  24,936
//   14.3, 15.0, 16.7, 19.6;  75,875 28.6, 32.9, 38.8, 47.1;  1.65 M 551, 655, 733, 818;
//   234,000 of a Q1 mesh, velocity gauge with complex scaling 106, 133, 211, 240
// 4 orbitals  6,234 nodes 7.0, 5.3, 5.2, 5.8;  24,936 9.3, 9.5, 9.8, 10.9;  49,872 13.7,
//   14.1, 15.5, 19.7;  75,875 16.8, 17.7, 19.0, 26.2;  1.65 M 273, 360, 360, 438
// 2 orbitals  6,234 nodes 7.0, 5.2, 4.9, 4.9;  49,872 11.0, 9.0, 9.7, 12.3;  75,875 13.1,
//   12.9, 13.4, 17.0 (in whole Arnoldi steps the same within the runs' spread);
//   151,750 18.8, 19.3, 21.1, 27.4;  1.65 M 173, 194, 217, 257 (velocity gauge 253, 235,
//   275, 307)
// 1 orbital   6,234 nodes 7.3, 5.8, 4.8, 4.6;  24,936 8.4, 5.9, 5.4, 6.0;  75,875 12.5,
//   10.4, 10.1, 11.4;  1.65 M 118, 127, 126, 159 (Q1 mesh as above 65, 26, 30, 36)
void launch_stencil_orb(const Batch& b, const double* u, const double* Ef, int diag_mode, const double* Upk,
                        const double* ginv, int mode, const double* lam, double* out, double* acc, hipStream_t s) {
  const int n = b.mx.n, L = n <= 1 ? 1 : n <= 2 ? 2 : n <= 4 ? 4 : 8;
  const int64_t lanes = b.mx.NE * L * b.ni;
  const bool few = lanes < (int64_t)1 << (L == 1 ? 14 : L == 2 ? 18 : 17);
  auto go = [&](auto f) { f(b, u, Ef, diag_mode, Upk, ginv, mode, lam, out, acc, s); };
  if (L == 1) few ? go(launch_orb_rows<1, 8>) : go(launch_orb_rows<1, 4>);
  else if (L == 2) few ? go(launch_orb_rows<2, 4>) : go(launch_orb_rows<2, 2>);
  else if (L == 4) few ? go(launch_orb_rows<4, 4>) : go(launch_orb_rows<4, 1>);
  else few ? go(launch_orb_rows<8, 4>) : go(launch_orb_rows<8, 1>);
}

// Masters: load value = acc_k + sum_h c_hk acc_h (transposed constraints), a
// master per 32 lanes (49 hanging rows on average at Q3, 180 at most; 8
// at Q1).  Sixteen lanes gathering whole orbital rows -> an orbital per lane:
// H2 (2,382 masters x 2 orbitals) 10.8 -> 4.8 us, 16 of it 26.6 -> 18.6 us, H2O
// (33,344 x 8) 60.9 -> 34.1 us.
template <int NP>
__global__ void __launch_bounds__(NT) k_ma_gather_orb(const DevMesh* __restrict__ dm, const double2* __restrict__ acc,
                                                      int mode, double2* __restrict__ out,
                                                      double2* __restrict__ ma_b) {
  INSTANCE;
  constexpr int LR = 32;
  const int n = d.n;
  const int64_t o = d.oE * n, om = d.oMa * n;
  const int lane = (int)(threadIdx.x & (LR - 1));
  const auto* ctp = gbl(d.ct_ptr);
  const XcdSweep sw = xcd_sweep(d.nMa, NT / LR);
  for (int64_t i = sw.start + threadIdx.x / LR; i < sw.end; i += sw.step) {
    const int64_t k = gbl(d.ma_dof)[i];
    double2 f = make_double2(0.0, 0.0);
    if (lane < n) f = ldg2(acc, o + k * n + lane);
    f = cadd(f, orb_row<NP, LR, NP == 8 ? 8 : 4>(d.ct_row, d.ct_w, ctp[i], ctp[i + 1], INT32_MAX, acc + o, n));
    if (lane < n) {
      if (mode == 0) out[o + k * n + lane] = f;
      else ma_b[om + i * n + lane] = f;
    }
  }
}

// Mass solve of a given load vector: non-masters 1/m, masters to ma_b.  out may be f.
__global__ void __launch_bounds__(NT) k_mass_direct(const DevMesh* __restrict__ dm, const double2* f, double2* out,
                                                    double2* __restrict__ ma_b) {
  INSTANCE;
  const int n = d.n;
  const int64_t total = d.N * n, o = d.oE * n, om = d.oMa * n;
  for (int64_t idx = (int64_t)blockIdx.x * NT + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * NT) {
    const int64_t k = idx / n;
    const int mi = gbl(d.ma_index)[k];
    if (mi < 0) out[o + idx] = cscale(gbl(d.inv_mass)[k], f[o + idx]);
    else ma_b[om + (int64_t)mi * n + (idx - k * n)] = f[o + idx];
  }
}

void launch_ma_gather_orb(const Batch& b, const double* acc, int mode, double* out, double* ma_b, hipStream_t s) {
  if (b.mx.nMa == 0) return;
  orb_dispatch(b.mx.n, [&](auto np) {
    hipLaunchKernelGGL(k_ma_gather_orb<np.value>, dim3(xcd_grid(b.mx.nMa, NT / 32, 65536), b.ni), dim3(NT), 0, s,
                       b.dm, (const double2*)acc, mode, (double2*)out, (double2*)ma_b);
  });
}

void launch_mass_direct(const Batch& b, const double* f, double* out, double* ma_b, hipStream_t s) {
  hipLaunchKernelGGL(k_mass_direct, dim3(nblocks(b.mx.N * b.mx.n, NT, 8192), b.ni), dim3(NT), 0, s, b.dm,
                     (const double2*)f, (double2*)out, (double2*)ma_b);
}

// --------------------------------------------------------------------------
// Assembled Poisson operator on the DoFs, K~ = C^T K_full C (CSR, built at
// set-up from the element line couplings): one dependent level per row
// (column index -> row of x), the hanging fill and the master gather folded
// into the matrix.  The matrix (about 12 B per entry, ~22 entries per row)
// is shared by all n^2 real columns.  L lanes per row, each owning V
// adjacent columns (16-byte loads for V >= 2); fused p.q partials.  x, q
// over extended rows (batch offset oE).
//
// Row lengths are very uneven: the masters of hanging nodes carry the
// constrained neighbourhood (up to several hundred entries against a median
// near 13).  Left to L lanes, such a row would keep its workgroup waiting
// for hundreds of dependent loads.  So the first `nlb` workgroups take the
// rows longer than KT_LONG, one row at a time per workgroup with all its
// NT / L lane groups splitting the entries and an LDS reduction; the other
// workgroups sweep the remaining rows.
// --------------------------------------------------------------------------
// Operator pass modes: the CG's operator pass on the preconditioned residual z
// (SP_CG); the residual r - K x
// (SP_RES: of a CG start, and the one that the restriction to the next
// multigrid level reads); and the Chebyshev smoothing passes of the multigrid
// cycle on the finest level:
// SP_CHEB0 runs the first two steps from z = 0 (its operand s0 D^-1 r is
// formed on the fly), SP_CHEB runs one step on a given z into another array.
// SP_CHEB_RZ is the second SP_CHEB step with r.z accumulated for the
// multigrid-preconditioned CG.
enum { SP_CG = 1, SP_CHEB0 = 2, SP_CHEB = 3, SP_CHEB_RZ = 4, SP_RES = 5 };

// Arrays of a pass beside its operand: w = K z of the CG's pass, double
// whatever z is; full: the operand of SP_RES is over full rows, and q holds r
// before the pass (the residual of a CG start, in place).
struct PassExtra {
  double* w;
  int full;
};

// Value of the operand at row j, columns c0 .. c0+V: x itself; (SP_CHEB0) beta
// D^-1_j x_j (x = r, beta = s0).
// T: storage type of the operand arrays (double; float for the finest-level
// multigrid arrays of Poisson schedule bit 6).  Arithmetic is in double.
template <int V, int MODE, class T>
__device__ __forceinline__ void operand_row(const __attribute__((address_space(1))) T* xg,
                                            const __attribute__((address_space(1))) double* dinv, const double* beta,
                                            int64_t j, int ld, int c0, double* out) {
  load_vals<V>(xg + j * ld + c0, out);  // 16-byte loads (ncol and c0 multiples of V)
  if constexpr (MODE == SP_CHEB0) {
    const double dj = dinv[j];
#pragma unroll
    for (int v = 0; v < V; ++v) out[v] = beta[v] * dj * out[v];
  }
}

// y += sum over entries t = beg, beg + stride, ... < end of val[t] operand(col[t]);
// four entries per round with all their loads issued together.  Past the end
// the index is clamped to the row's last entry (every row holds its diagonal)
// and the coefficient zeroed, so the loads need no branch.
template <int V, int MODE, class T>
__device__ __forceinline__ void spmv_row_part(const DevMesh& d, const T* __restrict__ x, const double* beta, int ld,
                                              int c0, int beg, int end, int stride, double* y) {
  const auto* kcol = gbl(d.kt_col);
  const auto* kval = gbl(d.kt_val);
  const auto* kvalf = gbl(d.kt_valf);   // the preconditioner's float passes read the float copy, the CG's own pass the doubles
  const auto* xg = gbl(x);
  const auto* dinv = gbl(d.kdiag_inv);
  for (int t = beg; t < end; t += 4 * stride) {
    double av[4];
    double xv[4][V];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int tt = t + u * stride;
      const int tc = tt < end ? tt : end - 1;
      const int64_t j = kcol[tc];
      double a;
      if constexpr (std::is_same<T, float>::value && MODE != SP_CG) a = kvalf[tc];
      else a = kval[tc];
      av[u] = tt < end ? a : 0.0;
      operand_row<V, MODE, T>(xg, dinv, beta, j, ld, c0, xv[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int v = 0; v < V; ++v) y[v] += av[u] * xv[u][v];
  }
}

// Row i done, y = (K operand)_i.  SP_CG: w_i = y and the z.w partial.
// Chebyshev passes (x: the operand's source, pprev = r, pout = z out, q = d,
// cf = the instance's coefficients s0, c1, c2; step k of SP_CHEB, step 1 for
// SP_CHEB_RZ):
//   SP_CHEB0: d0 = s0 D^-1 r, d = c1 d0 + c2 D^-1 (r - y), z = d0 + d (d not
//             stored when bit 8 of k is set: no further step reads it);
//   SP_CHEB:  d = c1 d + c D^-1 (r - y) (k = 0: c1 d dropped, c = s0; else
//             c1, c = c2 of step k), z = x + d; SP_CHEB_RZ also the r.z
//             partial (in pq), its step being k >> 4 (its slot k & 15); it is
//             the last step of a smoothing, so d is not stored.
// cf: s0, then (c1, c2) of each step from 1 on.
// SP_RES (x = z, pprev = r; ex.full: r in q): q_i = r_i - y.
template <int V, int MODE, class T>
__device__ __forceinline__ void spmv_store(const DevMesh& d, T* __restrict__ q, T* __restrict__ pout,
                                           const T* __restrict__ x, const T* __restrict__ pprev,
                                           const double* beta, int64_t i, int ld, int c0, const double* y,
                                           double* pq, const double* cf, int k, const PassExtra& ex) {
  const auto* dinv = gbl(d.kdiag_inv);
  if constexpr (MODE == SP_RES) {
    double rv[V];
    load_vals<V>(gbl(ex.full ? (const T*)q : pprev) + i * ld + c0, rv);
    T* qo = q + i * ld + c0;
#pragma unroll
    for (int v = 0; v < V; ++v) qo[v] = (T)(rv[v] - y[v]);
  } else if constexpr (MODE == SP_CHEB0 || MODE == SP_CHEB || MODE == SP_CHEB_RZ) {
    const int step = MODE == SP_CHEB_RZ ? k >> 4 : k;
    const double di = dinv[i];
    double rv[V], xv[V], dv[V];
    load_vals<V>(gbl(pprev) + i * ld + c0, rv);
    if constexpr (MODE != SP_CHEB0) {
      load_vals<V>(gbl(x) + i * ld + c0, xv);
      if (step > 0) load_vals<V>(gbl((const T*)q) + i * ld + c0, dv);
    }
    T* qo = q + i * ld + c0;
    T* po = pout + i * ld + c0;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      if constexpr (MODE == SP_CHEB0) {
        const double d0 = cf[0] * di * rv[v];
        const double dn = cf[1] * d0 + cf[2] * di * (rv[v] - y[v]);  // step 1
        if (!(k & 256)) qo[v] = (T)dn;
        po[v] = (T)(d0 + dn);
      } else {
        const double dn = (step > 0 ? cf[2 * step - 1] * dv[v] + cf[2 * step] * di * (rv[v] - y[v])
                                    : cf[0] * di * (rv[v] - y[v]));
        const double zn = xv[v] + dn;
        if constexpr (MODE != SP_CHEB_RZ) qo[v] = (T)dn;
        po[v] = (T)zn;
        if constexpr (MODE == SP_CHEB_RZ) pq[v] += rv[v] * zn;
      }
    }
  } else {
    double zi[V];
    operand_row<V, MODE, T>(gbl(x), dinv, beta, i, ld, c0, zi);
    auto* wo = gblw(ex.w) + i * ld + c0;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      wo[v] = y[v];
      pq[v] += zi[v] * y[v];
    }
  }
}

// The sums over g < groups of lds[g ncol + c] into lds[c], c < ncol (a tree;
// every thread of the workgroup calls it, threadIdx.x = g ncol + c).
__device__ __forceinline__ void col_tree(double* lds, int groups, int ncol) {
  int h = 1;
  while (2 * h < groups) h *= 2;
  const int g = (int)threadIdx.x / ncol;
  for (; h > 0; h >>= 1) {
    __syncthreads();
    if (g < h && g + h < groups) lds[threadIdx.x] += lds[threadIdx.x + h * ncol];
  }
  __syncthreads();
}

// lds[c] = sum over the rows w of part[w][c], c < nc, by one workgroup.
__device__ __forceinline__ void fold_cols(const double* __restrict__ part, int rows, int nc, double* lds) {
  const int per = NT / nc, g = (int)threadIdx.x / nc, c = (int)threadIdx.x - g * nc;
  const auto* pg = gbl(part);
  double s = 0.0;
  if (g < per)
    for (int w = g; w < rows; w += 8 * per) {
      double t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int ww = w + u * per;
        const double v = pg[(ww < rows ? ww : w) * nc + c];
        t[u] = ww < rows ? v : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) s += t[u];
    }
  lds[threadIdx.x] = s;
  col_tree(lds, per, nc);
}
// Largest number of partial sums that the launch that needs them folds itself:
// each of its workgroups reads them (64 KB from L2), which costs less than a
// launch; more are folded by k_fold_parts.  64 iterations of a solve with the
// bound at half, once, twice and four times this: 66,635 rows x 16 columns 3.35,
// 3.32, 3.36 and 3.54 ms; 4,394 x 25 3.53, 3.54, 3.62 and 3.62; x 64 2.87, 2.87,
// 2.87 and 3.08.
constexpr int64_t FOLD_MAX = 8192;

// Columns [col0, col0 + nc) of arrays with ld columns per row, col0 = blockIdx.z * nc
// (nc = ld without column blocking).  SELL: the short rows come from the
// sliced-ELL copy, a wave taking 64 / L slots of one slice (one width for all
// its rows), so each round of entries is read as consecutive words.
// MODE: SP_*; red: the CG accumulators ([ni][RED_SLOTS][ld]); k: the CG
// iteration (SP_CG), the smoothing step (SP_CHEB) or the r.z slot (SP_CHEB0 clears it, SP_CHEB_RZ
// accumulates into slot k & 15 at step k >> 4).
template <int L, int V, int MODE, bool SELL, class T>
__global__ void __launch_bounds__(NT) k_spmv_poisson(const DevMesh* __restrict__ dm, const T* __restrict__ x,
                                                     const T* __restrict__ pprev, T* __restrict__ pout,
                                                     int ld, int nc, T* __restrict__ q, int nlb,
                                                     double* __restrict__ red, int k, double* __restrict__ part,
                                                     PassExtra ex) {
  constexpr bool CG = MODE == SP_CG;
  INSTANCE;
  if (d.cg_done && *d.cg_done) return;  // converged instance of a batch CG (batches take no partials)
  __shared__ double lds[NT * V];
  // column block: blockIdx.z, or with schedule bit 7 the XCD's (xcd_sweep_cols;
  // the grid then runs all column blocks along x)
  const int nb_col = ld / nc;
  const bool aff = (d.sched_poi & 128) && nb_col > 1 && N_XCD % nb_col == 0;
  const int col0 = (aff ? ((int)blockIdx.x % N_XCD) % nb_col : (int)blockIdx.z) * nc;
  // one workgroup per column block clears the slots below (workgroup 0 of the
  // block's z slice; with bit 7 workgroups 0 .. nb_col - 1, one per block)
  const bool first_wg = aff ? (int)blockIdx.x < nb_col : blockIdx.x == 0;
  x += (MODE == SP_RES && ex.full ? d.oF : d.oE) * ld + col0;
  q += d.oE * ld + col0;
  pprev += d.oE * ld + col0;
  pout += d.oE * ld + col0;
  if (CG) ex.w += d.oE * ld + col0;
  double cf[2 * MG_MAX_DEG - 1];
#pragma unroll
  for (int j = 0; j < 2 * MG_MAX_DEG - 1; ++j) cf[j] = d.mgc[j];
  red += (int64_t)blockIdx.y * RED_SLOTS * ld + col0;
  const int lane = (int)(threadIdx.x & (L - 1));
  const int c0 = lane * V;
  const bool col_ok = c0 < nc;
  double beta[V];   // s0 for SP_CHEB0
#pragma unroll
  for (int v = 0; v < V; ++v) beta[v] = MODE == SP_CHEB0 ? cf[0] : 0.0;
  double pq[V];
#pragma unroll
  for (int v = 0; v < V; ++v) pq[v] = 0.0;
  if ((int)blockIdx.x < nlb) {
    // long rows: one per wave at a time, its 64 / L lane groups splitting the
    // entries, combined by shuffles (no workgroup barrier)
    constexpr int SEG = 64 / L;
    const int wave = threadIdx.x >> 6, seg = (threadIdx.x & 63) / L;
    // the long-row workgroups of this column block: all of them, or with column
    // blocks bound to XCDs those on this XCD's group (index gi of ng)
    int gi = (int)blockIdx.x, ng = nlb;
    if (aff) {
      const int G = N_XCD / nb_col;
      gi = ((int)blockIdx.x / N_XCD) * G + ((int)blockIdx.x % N_XCD) / nb_col;
      ng = nlb / N_XCD * G;
    }
    for (int64_t lr = (int64_t)gi * (NT / 64) + wave; lr < d.n_long; lr += (int64_t)ng * (NT / 64)) {
      const int64_t i = gbl(d.kt_long)[lr];
      const int beg = gbl(d.kt_ptr)[i], end = gbl(d.kt_ptr)[i + 1];
      double y[V];
#pragma unroll
      for (int v = 0; v < V; ++v) y[v] = 0.0;
      if (col_ok) spmv_row_part<V, MODE, T>(d, x, beta, ld, c0, beg + seg, end, SEG, y);
#pragma unroll
      for (int off = L; off < 64; off <<= 1)
#pragma unroll
        for (int v = 0; v < V; ++v) y[v] += __shfl_xor(y[v], off, 64);
      if (seg == 0 && col_ok) spmv_store<V, MODE, T>(d, q, pout, x, pprev, beta, i, ld, c0, y, pq, cf, k, ex);
    }
  } else if constexpr (SELL) {
    constexpr int R = 64 / L;  // slots per wave
    const int wave = threadIdx.x >> 6, slot_in = (threadIdx.x & 63) / L;
    const XcdSweep sw =
        aff ? xcd_sweep_cols(d.n_slices * L, NT / 64, nb_col, (int)blockIdx.x - nlb, (int)gridDim.x - nlb)
            : xcd_sweep(d.n_slices * L, NT / 64, d.sched_poi & 1, (int)blockIdx.x - nlb, (int)gridDim.x - nlb);
    const auto* sptr = gbl(d.sell_ptr);
    const auto* srow = gbl(d.sell_row);
    const auto* scol = gbl(d.sell_col);
    const auto* sval = gbl(d.sell_val);
    const auto* svalf = gbl(d.sell_valf);   // as in spmv_row_part
    const auto* xg = gbl(x);
    const auto* dinv = gbl(d.kdiag_inv);
    for (int64_t u = sw.start + wave; u < sw.end; u += sw.step) {
      const int64_t sl = u / L;
      const int slot = (int)(u - sl * L) * R + slot_in;
      const int i = srow[sl * SELL_H + slot];
      if (i < 0 || !col_ok) continue;
      const int base = sptr[sl], width = (sptr[sl + 1] - base) / SELL_H;
      double y[V];
#pragma unroll
      for (int v = 0; v < V; ++v) y[v] = 0.0;
      for (int t = 0; t < width; t += 4) {
        double av[4];
        double xv[4][V];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const int e = base + (t + h) * SELL_H + slot;
          if constexpr (std::is_same<T, float>::value && MODE != SP_CG) av[h] = svalf[e];
          else av[h] = sval[e];
          operand_row<V, MODE, T>(xg, dinv, beta, (int64_t)scol[e], ld, c0, xv[h]);
        }
#pragma unroll
        for (int h = 0; h < 4; ++h)
#pragma unroll
          for (int v = 0; v < V; ++v) y[v] += av[h] * xv[h][v];
      }
      spmv_store<V, MODE, T>(d, q, pout, x, pprev, beta, i, ld, c0, y, pq, cf, k, ex);
    }
  } else {
    const XcdSweep sw = aff ? xcd_sweep_cols(d.N, NT / L, nb_col, (int)blockIdx.x - nlb, (int)gridDim.x - nlb)
                            : xcd_sweep(d.N, NT / L, d.sched_poi & 1, (int)blockIdx.x - nlb, (int)gridDim.x - nlb);
    for (int64_t i = sw.start + threadIdx.x / L; i < sw.end; i += sw.step) {
      if (!col_ok) continue;
      const int beg = gbl(d.kt_ptr)[i], end = gbl(d.kt_ptr)[i + 1];
      if (nlb > 0 && end - beg > KT_LONG) continue;  // taken by the long-row workgroups
      double y[V];
#pragma unroll
      for (int v = 0; v < V; ++v) y[v] = 0.0;
      spmv_row_part<V, MODE, T>(d, x, beta, ld, c0, beg, end, 1, y);
      spmv_store<V, MODE, T>(d, q, pout, x, pprev, beta, i, ld, c0, y, pq, cf, k, ex);
    }
  }
  if constexpr (MODE == SP_CHEB0 || MODE == SP_CHEB || MODE == SP_RES) {
    if (MODE == SP_CHEB0 && first_wg && threadIdx.x < (unsigned)nc) red[(k & 255) * ld + threadIdx.x] = 0.0;
    return;
  }
  // z.w (r.z for SP_CHEB_RZ) of the workgroup: shuffles over the rows of each wave, then 4 waves
#pragma unroll
  for (int off = L; off < 64; off <<= 1)
#pragma unroll
    for (int v = 0; v < V; ++v) pq[v] += __shfl_xor(pq[v], off, 64);
  if ((threadIdx.x & 63) < (unsigned)L)
#pragma unroll
    for (int v = 0; v < V; ++v) lds[(threadIdx.x >> 6) * (L * V) + lane * V + v] = col_ok ? pq[v] : 0.0;
  __syncthreads();
  if (threadIdx.x < (unsigned)nc) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) sum += lds[w * (L * V) + threadIdx.x];
    if (part) {
      part[(int64_t)blockIdx.x * nc + threadIdx.x] = sum;  // folded by the next launch or by k_fold_parts
    } else {
      // r.z or z.w of this instance and column
      atomicAdd(red + (MODE == SP_CHEB_RZ ? (k & 15) : RED_PQ + k % 2) * ld + threadIdx.x, sum);
    }
    if (CG && first_wg) {  // clear what the update pass of this iteration accumulates into
      red[(RED_RZ + (k + 1) % 3) * ld + threadIdx.x] = 0.0;
      red[(RED_RR + k % 2) * ld + threadIdx.x] = 0.0;
    }
  }
}

// dst[c] += sum over the rows workgroups w of part[w][c] (one instance): the
// per-workgroup sums of an operator pass, added with a few hundred atomics
// where the pass itself would issue one per workgroup and column, all on the
// same nc addresses.  Bound by latency: eight loads in flight a thread (one after
// the other: 280 sums x 36 columns 6.7 -> 2.9 us).
__global__ void __launch_bounds__(NT) k_fold_parts(const double* __restrict__ part, int rows, int nc,
                                                   double* __restrict__ dst) {
  __shared__ double lds[NT];
  const int per = NT / nc, step = (int)gridDim.x * per;
  const int g = (int)threadIdx.x / nc, c = (int)threadIdx.x - g * nc;
  const auto* pg = gbl(part);
  double s = 0.0;
  if (g < per)
    for (int w = (int)blockIdx.x * per + g; w < rows; w += 8 * step) {
      double t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int ww = w + u * step;
        const double v = pg[(int64_t)(ww < rows ? ww : w) * nc + c];
        t[u] = ww < rows ? v : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) s += t[u];
    }
  lds[threadIdx.x] = s;
  col_tree(lds, per, nc);
  if (threadIdx.x < (unsigned)nc) atomicAdd(dst + threadIdx.x, lds[threadIdx.x]);
}

// Workgroups reserved for the long rows when schedule bit 2 or 5 is set:
// about two rows per wave, a multiple of 8 (so the XCD of the sweeping
// workgroups is unchanged).
static int long_row_blocks(const Batch& b) {
  if (b.mx.n_long == 0 || !(b.mx.sched_poi & (4 | 32))) return 0;
  const int64_t nb = std::min<int64_t>((b.mx.n_long + 2 * (NT / 64) - 1) / (2 * (NT / 64)), 2048);
  return (int)((nb + N_XCD - 1) / N_XCD * N_XCD);
}

// Set by the timed operator pass: the end event, recorded right after the pass
// kernel and before its fold, so the event pair spans that kernel alone.
static thread_local hipEvent_t t_pass_end = nullptr;

// Returns the number of partial sums per column left for the next launch to
// fold (0: the sums are in red).
template <int L, int V, int MODE, class T>
static int launch_spmv_m(const Batch& b, const T* x, const T* pprev, T* pout, int ld, int nc, T* q, double* red,
                         int k, const PassExtra& ex, hipStream_t s) {
  // schedule bit 7 with column blocks: the blocks ride along x, bound to XCDs
  // (the kernel takes the column block from the XCD), each block the whole sweep
  const int nbc = ld / nc;
  const bool sell = b.mx.sched_poi & 32;
  auto go = [&](const dim3& g, int nlb, double* part) {
    if (sell)
      hipLaunchKernelGGL((k_spmv_poisson<L, V, MODE, true, T>), g, dim3(NT), 0, s, b.dm, x, pprev, pout, ld, nc, q,
                         nlb, red, k, part, ex);
    else
      hipLaunchKernelGGL((k_spmv_poisson<L, V, MODE, false, T>), g, dim3(NT), 0, s, b.dm, x, pprev, pout, ld, nc, q,
                         nlb, red, k, part, ex);
    if (t_pass_end) (void)hipEventRecord(t_pass_end, s);
  };
  const int sweep = sell ? xcd_grid(b.mx.n_slices * L, NT / 64, b.mx.grid_poi) : xcd_grid(b.mx.N, NT / L, b.mx.grid_poi);
  if ((b.mx.sched_poi & 128) && nbc > 1 && N_XCD % nbc == 0) {
    const int nlb = long_row_blocks(b) * nbc;
    go(dim3(nlb + sweep * nbc, b.ni, 1), nlb, nullptr);
    return 0;
  }
  const int nlb = long_row_blocks(b);
  const int gx = nlb + sweep;
  // one instance: per-workgroup sums to a partial buffer, folded by the launch
  // that needs them or, where they are many, by one of their own
  double* part = nullptr;
  bool later = false;
  if constexpr (MODE == SP_CG || MODE == SP_CHEB_RZ)
    if (b.spart && b.ni == 1 && nc == ld && (int64_t)gx * nc <= b.spart_cap) {
      later = (int64_t)gx * nc <= FOLD_MAX;
      part = later && MODE == SP_CHEB_RZ ? b.spart + b.spart_cap : b.spart;   // both are folded by the update pass
    }
  go(dim3(gx, b.ni, nbc), nlb, part);
  if (later) return gx;
  if (part) {
    const int slot = MODE == SP_CHEB_RZ ? (k & 15) : RED_PQ + k % 2;
    const int fb = (int)std::max<int64_t>(1, std::min<int64_t>(256, (int64_t)gx / (NT / nc * 8)));
    hipLaunchKernelGGL(k_fold_parts, dim3(fb), dim3(NT), 0, s, part, gx, nc, red + (int64_t)slot * ld);
  }
  return 0;
}
template <int L, int V, class T>
static int launch_spmv_t(const Batch& b, const T* x, const T* pprev, T* pout, int ld, int nc, T* q, double* red,
                         int mode, int k, const PassExtra& ex, hipStream_t s) {
  switch (mode) {
    case SP_CG: return launch_spmv_m<L, V, SP_CG, T>(b, x, pprev, pout, ld, nc, q, red, k, ex, s);
    case SP_CHEB0: return launch_spmv_m<L, V, SP_CHEB0, T>(b, x, pprev, pout, ld, nc, q, red, k, ex, s);
    case SP_CHEB: return launch_spmv_m<L, V, SP_CHEB, T>(b, x, pprev, pout, ld, nc, q, red, k, ex, s);
    case SP_RES: return launch_spmv_m<L, V, SP_RES, T>(b, x, pprev, pout, ld, nc, q, red, k, ex, s);
    default: return launch_spmv_m<L, V, SP_CHEB_RZ, T>(b, x, pprev, pout, ld, nc, q, red, k, ex, s);
  }
}

// One operator pass in the given mode over all columns.
// Schedule bit 1 (column blocking): with 32 or more columns in multiples of 16,
// grid.z runs over blocks of 16 columns, so a row slice is 128 B and the band of
// neighbour rows a sweep touches stays in L2 (the matrix is read once per block).
template <class T>
static int launch_spmv_mode(const Batch& b, const T* x, const T* pprev, T* pout, int ncol, T* q, double* red,
                            int mode, int k, hipStream_t s, const PassExtra& ex) {
  if ((b.mx.sched_poi & 2) && ncol >= 32 && ncol % 16 == 0)
    return launch_spmv_t<4, 4, T>(b, x, pprev, pout, ncol, 16, q, red, mode, k, ex, s);
  if (ncol % 4 == 0 && ncol > 4) {  // 4 columns per lane (two 16-byte loads; one for float)
    if (ncol <= 16) return launch_spmv_t<4, 4, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
    if (ncol <= 32) return launch_spmv_t<8, 4, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
    return launch_spmv_t<16, 4, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
  }
  if (ncol % 2 == 0) {  // column pairs
    if (ncol <= 4) return launch_spmv_t<2, 2, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
    if (ncol <= 8) return launch_spmv_t<4, 2, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
    if (ncol <= 16) return launch_spmv_t<8, 2, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
    if (ncol <= 32) return launch_spmv_t<16, 2, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
    return launch_spmv_t<32, 2, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
  }
  if (ncol <= 1) return launch_spmv_t<1, 1, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
  if (ncol <= 2) return launch_spmv_t<2, 1, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
  if (ncol <= 4) return launch_spmv_t<4, 1, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
  if (ncol <= 8) return launch_spmv_t<8, 1, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
  if (ncol <= 16) return launch_spmv_t<16, 1, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
  if (ncol <= 32) return launch_spmv_t<32, 1, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
  return launch_spmv_t<64, 1, T>(b, x, pprev, pout, ncol, ncol, q, red, mode, k, ex, s);
}
static PassExtra no_extra(int full = 0) { return PassExtra{nullptr, full}; }

// --------------------------------------------------------------------------
// Jacobi-preconditioned CG, all columns of all instances at once with their
// own alpha and beta.  Scalars sc[i][slot][c] (SC_*) and red[i][slot][c] (RED_*)
// in kernels.hpp.
// --------------------------------------------------------------------------
// One CG iteration is two launches beside its preconditioner: the operator
// pass, w = K z with z.w, and the vector pass,
//   beta = r.z / (r.z)_old, eta = z.w - beta^2 eta_old, alpha = r.z / eta,
//   p = z + beta p, q = w + beta q, x += alpha p, r -= alpha q, r.r
// (Chronopoulos and Gear 1989): q is K p by its recurrence and eta is p.q, as
// the directions are K-orthogonal, so the operator pass takes z and needs no
// scalar of the iteration.  It gathers z (float rows where the multigrid
// level keeps floats) instead of p, in whatever row order it runs, while
// every vector is swept once, in order.  eta is taken from z.w alone (a restart,
// beta = 0) where the subtraction leaves less than a thousandth of z.w, so a
// column at its rounding floor cannot take a step of arbitrary length: a solve leaves
// a third of it or more (Jacobi, five meshes, to 1e-13), and at a thousandth alpha
// would keep 13 digits, with a float z, orthogonal to the last residual to 1e-7, four.
// Solves to between 1e-8 and 3e-16 take the iterations that the form with p.q summed
// takes, to the same distance from the direct solution.
// x takes two iterations' terms at once, every second iteration (one instance;
// the instances of a batch stop at different iterations).
// Against a direction pass, an operator pass on p and an update pass with
// their sums folded by launches of their own: H2O (1.5 M rows x 64 columns,
// float z) 2.52 -> 2.30 ms per iteration, 16 H2 (1.16 M x 4) 284 -> 217 us, Q1 water
// (0.2 M x 64) 255 -> 212 us, H2 (66,635 x 4) 39 -> 27 us.  With the vector
// updates in the operator pass itself H2O takes 2.22 ms, but 16 H2 382 us: with
// few columns the rows of a wave, sorted by length, lie apart.
// The accumulators rotate (rz over three slots, z.w, eta and r.r over two), and
// each pass clears only slots that no workgroup of the same launch reads, so
// no launch overwrites a value its own workgroups use.

// The vector pass.  JAC: z = D^-1 r, formed here and, of the new r, written for the
// next operator pass (zj); r.D^-1 r of the new r is accumulated for the next
// iteration.  With D^-1 gathered beside r in the operator pass instead of the store
// here, that pass waited for one more dependent load an entry: 66,635 rows x 4
// columns 20.4 -> 16.5 us (this pass 12.0 -> 12.4), four times that in a batch 48.1 ->
// 40.2 (19.2 -> 19.9), 4,394 x 25 43.2 -> 37.6 (9.4 both), 66,635 x 64 in blocks of 16
// columns 197 -> 149 (53.6 -> 60.3).
// xmode 0: x left for the next pass; 1: x += alpha p;
// 2: also the previous iteration's term.  zw_rows, rz_rows > 0: z.w and r.z are
// folded here from the partial sums of the passes that formed them.
// A thread takes one column and U rows at a time, all their loads in flight
// before the first store.
template <class Z, bool JAC, int U>
__global__ void __launch_bounds__(NT) k_cg_vectors(const DevMesh* __restrict__ dm, double* __restrict__ x,
                                                   double* __restrict__ r, const Z* __restrict__ z,
                                                   double* __restrict__ p, const double* __restrict__ w,
                                                   double* __restrict__ q, int ncol, double* __restrict__ red, int k,
                                                   float* __restrict__ rf, double* __restrict__ zj, int xmode,
                                                   const double* __restrict__ zw_part, int zw_rows,
                                                   const double* __restrict__ rz_part, int rz_rows) {
  INSTANCE;
  if (d.cg_done && *d.cg_done) return;
  __shared__ double lds[2 * NT];
  x += d.oF * ncol;
  if (rf) rf += d.oE * ncol;
  r += d.oE * ncol;
  if (JAC) zj += d.oE * ncol;
  else z += d.oE * ncol;
  p += d.oE * ncol;
  w += d.oE * ncol;
  q += d.oE * ncol;
  red += (int64_t)blockIdx.y * RED_SLOTS * ncol;
  const int groups = NT / ncol;
  const int g = threadIdx.x / ncol, c = threadIdx.x - g * ncol;
  const bool act = g < groups;
  const auto* dinv = gbl(d.kdiag_inv);
  if (zw_rows > 0) fold_cols(zw_part, zw_rows, ncol, lds);
  if (rz_rows > 0) fold_cols(rz_part, rz_rows, ncol, lds + NT);
  double rz = 0.0, rr = 0.0;
  if (act) {
    const double ga = rz_rows > 0 ? lds[NT + c] : red[(RED_RZ + k % 3) * ncol + c];
    const double zw = zw_rows > 0 ? lds[c] : red[(RED_PQ + k % 2) * ncol + c];
    double be = 0.0, eta = zw, alp = 0.0;
    if (k > 0) {
      const double gp = red[(RED_RZ + (k + 2) % 3) * ncol + c], ep = red[(RED_ETA + (k + 1) % 2) * ncol + c];
      be = gp != 0.0 ? ga / gp : 0.0;
      alp = (ep != 0.0 && gp != 0.0) ? gp / ep : 0.0;
      eta = zw - be * be * ep;
      if (!(eta > 1e-3 * zw)) {
        be = 0.0;
        eta = zw;
      }
    }
    const double al = (eta != 0.0 && ga != 0.0) ? ga / eta : 0.0;
    if (blockIdx.x == 0 && g == 0) {
      if (rz_rows > 0) red[(RED_RZ + k % 3) * ncol + c] = ga;
      red[(RED_ETA + k % 2) * ncol + c] = eta;
      red[(RED_PQ + (k + 1) % 2) * ncol + c] = 0.0;  // for the next operator pass
    }
    const int64_t step = (int64_t)gridDim.x * groups;
    for (int64_t kk = (int64_t)blockIdx.x * groups + g; kk < d.N; kk += U * step) {
      double ro[U], wi[U], zi[U], po[U], qo[U], xo[U], di[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t row = kk + u * step < d.N ? kk + u * step : kk;   // past the end: the first row again, not stored
        const int64_t e = row * ncol + c;
        ro[u] = r[e];
        wi[u] = w[e];
        di[u] = JAC ? dinv[row] : 0.0;
        zi[u] = JAC ? di[u] * ro[u] : (double)z[e];
        po[u] = k > 0 ? p[e] : 0.0;
        qo[u] = k > 0 ? q[e] : 0.0;
        xo[u] = xmode ? x[e] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u > 0 && kk + u * step >= d.N) break;
        const int64_t e = (kk + u * step) * ncol + c;
        const double pn = zi[u] + be * po[u], qn = wi[u] + be * qo[u];
        p[e] = pn;
        q[e] = qn;
        if (xmode) x[e] = xo[u] + (xmode == 2 ? alp * po[u] + al * pn : al * pn);
        const double rn = ro[u] - al * qn;
        r[e] = rn;
        if (rf) rf[e] = (float)rn;  // the finest multigrid level's float copy (Poisson schedule bit 6)
        if (JAC) {
          zj[e] = di[u] * rn;
          rz += rn * rn * di[u];
        }
        rr += rn * rn;
      }
    }
  }
  __syncthreads();
  lds[threadIdx.x] = act ? rr : 0.0;
  if (JAC) lds[NT + threadIdx.x] = act ? rz : 0.0;
  col_tree(lds, groups, ncol);
  if (JAC) col_tree(lds + NT, groups, ncol);
  if (threadIdx.x < (unsigned)ncol) {
    atomicAdd(red + (RED_RR + k % 2) * ncol + threadIdx.x, lds[threadIdx.x]);
    if (JAC) atomicAdd(red + (RED_RZ + (k + 1) % 3) * ncol + threadIdx.x, lds[NT + threadIdx.x]);
  }
}

// Initial rz, rr from the start partials (rz_0 into slot RED_RZ, r.r also
// into SC_RR); the other accumulators cleared.
__global__ void __launch_bounds__(NT) k_rz_start(const double* __restrict__ part, int64_t part_stride, int nblk,
                                                 int ncol, double* __restrict__ sc, double* __restrict__ red) {
  __shared__ double lds4[4];
  const int c = blockIdx.x;
  part += blockIdx.y * part_stride;
  sc += (int64_t)blockIdx.y * SC_SLOTS * ncol;
  red += (int64_t)blockIdx.y * RED_SLOTS * ncol;
  const double s = sum_partials(part, nblk, 2 * ncol, c, lds4);
  const double u = sum_partials(part, nblk, 2 * ncol, ncol + c, lds4);
  if (threadIdx.x == 0) {
    for (int slot = 0; slot < RED_SLOTS; ++slot) red[slot * ncol + c] = 0.0;
    red[RED_RZ * ncol + c] = s;
    sc[SC_RR * ncol + c] = u;
  }
}

// start: partial rz, rr of the first residual r (cold: x = 0).  x over full rows.
// z: null, or D^-1 r for the Jacobi CG's first operator pass.
__global__ void __launch_bounds__(NT) k_cg_start2(const DevMesh* __restrict__ dm, double* __restrict__ x,
                                                  const double* __restrict__ r, double* __restrict__ z, int ncol,
                                                  int warm, int64_t part_stride, double* __restrict__ part) {
  INSTANCE;
  __shared__ double lds[2 * NT];
  x += d.oF * ncol;
  r += d.oE * ncol;
  if (z) z += d.oE * ncol;
  const int groups = NT / ncol;
  const int g = threadIdx.x / ncol, c = threadIdx.x - g * ncol;
  const bool act = g < groups;
  double rz = 0.0, rr = 0.0;
  if (act)
    for (int64_t k = (int64_t)blockIdx.x * groups + g; k < d.N; k += (int64_t)gridDim.x * groups) {
      const int64_t e = k * ncol + c;
      const double rn = r[e];
      if (!warm) x[e] = 0.0;
      const double di = gbl(d.kdiag_inv)[k];
      if (z) z[e] = di * rn;
      rz += rn * rn * di;
      rr += rn * rn;
    }
  lds[threadIdx.x] = act ? rz : 0.0;
  lds[NT + threadIdx.x] = act ? rr : 0.0;
  col_tree(lds, groups, ncol);
  col_tree(lds + NT, groups, ncol);
  if (threadIdx.x < (unsigned)ncol) {
    double* pb = part + blockIdx.y * part_stride + (int64_t)blockIdx.x * 2 * ncol;
    pb[threadIdx.x] = lds[threadIdx.x];
    pb[ncol + threadIdx.x] = lds[NT + threadIdx.x];
  }
}

// Workgroups of the CG start and update passes: about 32 elements per thread,
// at least RED_BLOCKS (small meshes: few partial sums) and at most 2048 (eight
// per compute unit), so the passes over large meshes keep enough loads in flight.
static int cg_blocks(const Batch& b, int ncol) {
  const int64_t want = std::min<int64_t>(std::max<int64_t>(b.mx.N * ncol / (NT * 32), RED_BLOCKS), 2048);
  return nblocks(b.mx.N, NT / ncol, (int)want);
}

// An operator pass of the CG (one per iteration, and the residual of a warm
// start) with optional event timing on the launch stream.
template <class F>
static int timed_pass(PoissonWs& P, hipStream_t s, F&& pass) {
  const bool rec = P.ev && P.ev_used + 2 <= P.ev_cap;
  if (rec) {
    (void)hipEventRecord(P.ev[P.ev_used], s);
    t_pass_end = P.ev[P.ev_used + 1];
  }
  const int rows = pass();
  if (rec) {
    t_pass_end = nullptr;
    P.ev_used += 2;
  }
  return rows;
}
template <class T>
static int cg_pass(const Batch& b, PoissonWs& P, const T* z, int k, hipStream_t s) {
  return timed_pass(P, s, [&] {
    return launch_spmv_mode<T>(b, z, z, nullptr, P.ncol, nullptr, P.red, SP_CG, k, s, PassExtra{P.w, 0});
  });
}
// How the solution update of iteration k is taken (k_cg_vectors).
static int cg_xmode(const Batch& b, int k) { return b.ni > 1 ? 1 : (k % 2 ? 2 : 0); }

constexpr int CG_ROWS = 2;
template <class Z, bool JAC>
static void cg_vectors(const Batch& b, double* W, PoissonWs& P, const Z* z, float* rf, int zw_rows, int rz_rows, int k,
                       hipStream_t s) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(cg_blocks(b, P.ncol), b.ni), dim3(NT), 0, s, b.dm, W, P.r, z, P.p,
                       (const double*)P.w, P.q, P.ncol, P.red, k, rf, JAC ? P.acc : nullptr, cg_xmode(b, k), (const double*)b.spart, zw_rows,
                       (const double*)(b.spart ? b.spart + b.spart_cap : nullptr), rz_rows);
  };
  go(k_cg_vectors<Z, JAC, CG_ROWS>);
}
template <class Z>
static void cg_iteration(const Batch& b, double* W, PoissonWs& P, const Z* z, float* rf, int rz_rows, int k,
                         hipStream_t s) {
  const int rows = cg_pass<Z>(b, P, z, k, s);
  cg_vectors<Z, false>(b, W, P, z, rf, rows, rz_rows, k, s);
}
void launch_cg_iteration(const Batch& b, double* W, PoissonWs& P, const double* z, float* rf, int rz_rows, int k,
                         hipStream_t s) {
  cg_iteration(b, W, P, z, rf, rz_rows, k, s);
}
void launch_cg_iteration(const Batch& b, double* W, PoissonWs& P, const float* z, float* rf, int rz_rows, int k,
                         hipStream_t s) {
  cg_iteration(b, W, P, z, rf, rz_rows, k, s);
}
// One Jacobi-preconditioned iteration.
void launch_cg_step(const Batch& b, double* W, PoissonWs& P, hipStream_t s) {
  const int k = P.it;
  const int rows = cg_pass<double>(b, P, P.acc, k, s);
  cg_vectors<double, true>(b, W, P, nullptr, nullptr, rows, 0, k, s);
  P.it = k + 1;
}
// The solution update still open after `it` iterations: x += alpha p of the
// last one where it left its term to a next pass.
void launch_cg_finish(const Batch& b, double* W, PoissonWs& P, int it, hipStream_t s) {
  if (it > 0 && cg_xmode(b, it - 1) == 0)
    cg_xfinal(b.dm, b.ni, b.mx.N, P.ncol, W, P.p, P.red, RED_RZ + (it - 1) % 3, RED_ETA + (it - 1) % 2, s);
}

void launch_cg_start(const Batch& b, double* W, double* rhs_r, PoissonWs& P, int warm, hipStream_t s) {
  const int ncol = P.ncol;
  // warm: r = rhs - K x0, x0 = the DoF rows of W (full rows)
  if (warm)
    timed_pass(P, s, [&] {
      return launch_spmv_mode<double>(b, W, nullptr, nullptr, ncol, rhs_r, P.red, SP_RES, -1, s, no_extra(1));
    });
  const int nb = cg_blocks(b, ncol);
  hipLaunchKernelGGL(k_cg_start2, dim3(nb, b.ni), dim3(NT), 0, s, b.dm, W, rhs_r,
                     b.mx.sched_poi & 16 ? nullptr : P.acc, ncol, warm, P.part_stride, P.part);
  hipLaunchKernelGGL(k_rz_start, dim3(ncol, b.ni), dim3(NT), 0, s, P.part, P.part_stride, nb, ncol, P.sc, P.red);
  P.it = 0;
}

// Chebyshev smoothing on the finest multigrid level fused into the operator
// pass (the spmv_store comment gives the updates): the first two steps from
// zero (z, d from r), and one further step from zin into zout.
// t = r - K z on the finest level (the residual the restriction reads)
void launch_mg_resid(const Batch& b, const double* z, const double* r, double* t, int ncol, hipStream_t s) {
  launch_spmv_mode<double>(b, z, r, t, ncol, t, nullptr, SP_RES, -1, s, no_extra());
}
void launch_mg_resid_f(const Batch& b, const float* z, const float* r, float* t, int ncol, hipStream_t s) {
  launch_spmv_mode<float>(b, z, r, t, ncol, t, nullptr, SP_RES, -1, s, no_extra());
}
void launch_mg_cheb0(const Batch& b, const double* r, double* z, double* d, double* red, int rz_slot, int ncol,
                     hipStream_t s) {
  launch_spmv_mode(b, r, r, z, ncol, d, red, SP_CHEB0, rz_slot, s, no_extra());
}
int launch_mg_cheb_step(const Batch& b, const double* zin, const double* r, double* zout, double* d, double* red,
                         int ncol, int k, int rz_slot, hipStream_t s) {
  if (rz_slot >= 0)
    return launch_spmv_mode(b, zin, r, zout, ncol, d, red, SP_CHEB_RZ, rz_slot | (k << 4), s, no_extra());
  return launch_spmv_mode(b, zin, r, zout, ncol, d, red, SP_CHEB, k, s, no_extra());
}

// The same finest-level passes on float storage (Poisson schedule bit 6):
// operand, residual copy, corrections and directions in float, sums in
// double.  These passes are not event-timed (the timing slot holds the
// double passes of the CG itself).
void launch_mg_cheb0_f(const Batch& b, const float* r, float* z, float* d, double* red, int rz_slot, int ncol,
                       hipStream_t s) {
  launch_spmv_mode<float>(b, r, r, z, ncol, d, red, SP_CHEB0, rz_slot, s, no_extra());
}
int launch_mg_cheb_step_f(const Batch& b, const float* zin, const float* r, float* zout, float* d, double* red,
                           int ncol, int k, int rz_slot, hipStream_t s) {
  if (rz_slot >= 0)
    return launch_spmv_mode<float>(b, zin, r, zout, ncol, d, red, SP_CHEB_RZ, rz_slot | (k << 4), s, no_extra());
  return launch_spmv_mode<float>(b, zin, r, zout, ncol, d, red, SP_CHEB, k, s, no_extra());
}

// Convergence flags of a batch's multigrid CG (the host test of the same
// solve, on the device): after the update pass of iteration k an instance is
// done once every column's r.r is at most rtol^2 times its largest column's
// b.b.  Its r.r is then copied into the other r.r slot as well, so the final
// test reads a converged value whichever iteration the solve stops after,
// and its later CG and multigrid launches return at once.  One wave per
// instance (ncol <= 64).
__global__ void k_cg_done(const DevMesh* __restrict__ dm, const double* __restrict__ sc, double* __restrict__ red,
                          int ncol, int k, double rtol2) {
  INSTANCE;
  if (!d.cg_done || *d.cg_done) return;
  sc += (int64_t)blockIdx.y * SC_SLOTS * ncol;
  red += (int64_t)blockIdx.y * RED_SLOTS * ncol;
  const int c = threadIdx.x;
  double bb = c < ncol ? sc[SC_BB * ncol + c] : 0.0;
  for (int off = 32; off > 0; off >>= 1) bb = fmax(bb, __shfl_xor(bb, off, 64));
  const double rr = c < ncol ? red[(RED_RR + k % 2) * ncol + c] : 0.0;
  const bool ok = c >= ncol || rr <= rtol2 * bb;
  if (__all(ok)) {
    if (c < ncol) red[(RED_RR + (k + 1) % 2) * ncol + c] = rr;
    if (c == 0) *const_cast<int*>(d.cg_done) = 1;
  }
}
void launch_cg_done(const Batch& b, const PoissonWs& P, int k, double rtol, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_done, dim3(1, b.ni), dim3(64), 0, s, b.dm, P.sc, P.red, P.ncol, k, rtol * rtol);
}
__global__ void k_zero_int(int* __restrict__ x, int n) {
  for (int i = blockIdx.x * NT + threadIdx.x; i < n; i += gridDim.x * NT) x[i] = 0;
}
void launch_zero_int(int* x, int n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_zero_int, dim3(nblocks(n)), dim3(NT), 0, s, x, n);
}

__global__ void __launch_bounds__(NT) k_to_float(const double* __restrict__ x, float* __restrict__ y, int64_t nd) {
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < nd; i += (int64_t)gridDim.x * NT) y[i] = (float)x[i];
}
void launch_to_float(const double* x, float* y, int64_t nd, hipStream_t s) {
  if (nd > 0) hipLaunchKernelGGL(k_to_float, dim3(nblocks(nd, NT, 8192)), dim3(NT), 0, s, x, y, nd);
}

// y = a x + b y over nd doubles (a, b real)
__global__ void __launch_bounds__(NT) k_axpby(int64_t nd, double a, const double* __restrict__ x, double b,
                                              double* __restrict__ y) {
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < nd; i += (int64_t)gridDim.x * NT)
    y[i] = a * x[i] + b * y[i];
}
void launch_axpby(int64_t nd, double a, const double* x, double b, double* y, hipStream_t s) {
  if (nd > 0) hipLaunchKernelGGL(k_axpby, dim3(nblocks(nd, NT, 8192)), dim3(NT), 0, s, nd, a, x, b, y);
}

}  // namespace mh
