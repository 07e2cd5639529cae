// Host set-up of the geometric multigrid hierarchy for the pair Poisson
// operator: coarse meshes, their assembled operators, the interpolation
// between consecutive levels, smoother bounds and the dense coarsest inverse.
#include <algorithm>
#include <cmath>
#include <stdexcept>
#include <unordered_map>

#include "host.hpp"

namespace mh {

namespace {

uint64_t leaf_key(int l, int64_t i, int64_t j, int64_t k) {
  return ((uint64_t)l << 60) | ((uint64_t)i << 40) | ((uint64_t)j << 20) | (uint64_t)k;
}

// Leaf of mesh C containing point x (on a shared face any adjacent leaf does:
// the coarse function is continuous there).
int64_t locate(const Mesh& C, const std::unordered_map<uint64_t, int64_t>& leaves, const double* x) {
  for (int l = 0; l <= C.Lmax; ++l) {
    const int64_t n = (int64_t)C.nc << l;
    const double h = (C.hi - C.lo) / (double)n;
    int64_t ijk[3];
    for (int d = 0; d < 3; ++d) {
      int64_t t = (int64_t)std::floor((x[d] - C.lo) / h);
      ijk[d] = std::min<int64_t>(std::max<int64_t>(t, 0), n - 1);
    }
    auto it = leaves.find(leaf_key(l, ijk[0], ijk[1], ijk[2]));
    if (it != leaves.end()) return it->second;
  }
  return -1;
}

// Prolongation rows: for each DoF node of F, the coarse function's value there
// as a combination of C's DoFs.
void prolongation(const Mesh& F, const Mesh& C, MgLevel& out, Crew& crew) {
  std::unordered_map<uint64_t, int64_t> leaves;
  leaves.reserve(C.n_cells * 2);
  for (int64_t e = 0; e < C.n_cells; ++e)
    leaves[leaf_key(C.cell_level[e], C.cell_ijk[3 * e], C.cell_ijk[3 * e + 1], C.cell_ijk[3 * e + 2])] = e;
  const int P = C.P;
  const int64_t NEc = C.N + C.Nh;
  out.p_ptr.assign(F.N + 1, 0);
  struct Part {
    std::vector<int32_t> col;
    std::vector<double> val;
  };
  const int parts = crew.parts(2 * F.N * P * P * P);
  std::vector<Part> part(parts);
  crew.ranges(F.N, parts, [&](int c0, int64_t lo, int64_t hi) {
    Part& po = part[c0];
    std::vector<std::pair<int32_t, double>> row;   // sums by column, in order of first appearance
    for (int64_t i = lo; i < hi; ++i) {
      const double* x = &F.xyz[3 * i];
      const int64_t e = locate(C, leaves, x);
      if (e < 0) throw std::runtime_error("multigrid: fine node outside the coarse mesh");
      double w1[3][4];
      for (int d = 0; d < 3; ++d) {
        const double xi = 2.0 * (x[d] - C.cell_org[3 * e + d]) / C.cell_h[e] - 1.0;
        for (int a = 0; a < P; ++a) w1[d][a] = lagrange(C.gll.x, a, xi);
      }
      row.clear();
      auto add = [&](int64_t c, double w) {
        for (auto& r : row)
          if (r.first == c) {
            r.second += w;
            return;
          }
        row.push_back({(int32_t)c, w});
      };
      for (int c = 0; c < P; ++c)
        for (int b = 0; b < P; ++b)
          for (int a = 0; a < P; ++a) {
            const double w = w1[0][a] * w1[1][b] * w1[2][c];
            if (std::fabs(w) < 1e-15) continue;
            const int64_t nd = C.cell_nodes[(e * P + c) * P * P + b * P + a];
            if (nd < C.N) {
              add(nd, w);
            } else if (nd < NEc) {  // hanging: its constraint row (boundary masters carry zero)
              const int64_t h = nd - C.N;
              for (int64_t t = C.hang_ptr[h]; t < C.hang_ptr[h + 1]; ++t)
                if (C.hang_col[t] < C.N) add(C.hang_col[t], w * C.hang_w[t]);
            }
          }
      std::sort(row.begin(), row.end());
      const size_t beg = po.col.size();
      for (const auto& kv : row)
        if (std::fabs(kv.second) > 1e-14) {
          po.col.push_back(kv.first);
          po.val.push_back(kv.second);
        }
      out.p_ptr[i + 1] = (int32_t)(po.col.size() - beg);
    }
  });
  int64_t nnz = 0;
  for (int64_t i = 0; i < F.N; ++i) {
    nnz += out.p_ptr[i + 1];
    if (nnz >= INT32_MAX) throw std::runtime_error("multigrid: prolongation too large");
    out.p_ptr[i + 1] = (int32_t)nnz;
  }
  out.p_col.swap(part[0].col);
  out.p_val.swap(part[0].val);
  for (int c = 1; c < parts; ++c) {
    out.p_col.insert(out.p_col.end(), part[c].col.begin(), part[c].col.end());
    out.p_val.insert(out.p_val.end(), part[c].val.begin(), part[c].val.end());
  }
  // transpose
  const int64_t Nc = C.N;
  out.r_ptr.assign(Nc + 1, 0);
  for (int32_t c : out.p_col) out.r_ptr[c + 1]++;
  for (int64_t c = 0; c < Nc; ++c) out.r_ptr[c + 1] += out.r_ptr[c];
  out.r_col.assign(out.p_col.size(), 0);
  out.r_val.assign(out.p_col.size(), 0.0);
  std::vector<int32_t> fill(out.r_ptr.begin(), out.r_ptr.end() - 1);
  for (int64_t i = 0; i < F.N; ++i)
    for (int32_t t = out.p_ptr[i]; t < out.p_ptr[i + 1]; ++t) {
      const int32_t c = out.p_col[t];
      out.r_col[fill[c]] = (int32_t)i;
      out.r_val[fill[c]++] = out.p_val[t];
    }
}

// Largest eigenvalue of D^-1 K by power iteration (a fixed seed-free start).
double lambda_max(const MgLevel& L, Crew& crew) {
  std::vector<double> x(L.N), y(L.N);
  for (int64_t i = 0; i < L.N; ++i) x[i] = 1.0 + 0.5 * std::sin(0.7 * (double)i);
  const int parts = crew.parts((int64_t)L.k_col.size());
  double lam = 0.0, nrm = 1.0;
  for (int it = 0; it < 40; ++it) {
    crew.ranges(L.N, parts, [&](int, int64_t lo, int64_t hi) {
      for (int64_t i = lo; i < hi; ++i) {
        double s = 0.0;
        for (int32_t t = L.k_ptr[i]; t < L.k_ptr[i + 1]; ++t) s += L.k_val[t] * x[L.k_col[t]];
        y[i] = s * L.dinv[i];
      }
    });
    double yn = 0.0, xn = 0.0;
    for (int64_t i = 0; i < L.N; ++i) {
      yn += y[i] * y[i];
      xn += x[i] * x[i];
    }
    nrm = std::sqrt(yn);
    lam = nrm / std::sqrt(xn);
    for (int64_t i = 0; i < L.N; ++i) x[i] = y[i] / nrm;
  }
  return lam;
}

void take_operator(const OpHost& H, int64_t N, MgLevel& L) {
  L.N = N;
  L.k_ptr = H.kt_ptr;
  L.k_col = H.kt_col;
  L.k_val = H.kt_val;
  L.dinv = H.kdiag_inv;
}

// Tables of the cell-by-cell prolongation where mesh C has F's leaves at a lower
// degree: F's levels' cell_f, cell_c and C's hanging rows (into the level of C).
void cell_transfer(const Mesh& F, const Mesh& C, MgLevel& lf, MgLevel& lc) {
  std::unordered_map<uint64_t, int64_t> leaves;
  leaves.reserve(C.n_cells * 2);
  for (int64_t e = 0; e < C.n_cells; ++e)
    leaves[leaf_key(C.cell_level[e], C.cell_ijk[3 * e], C.cell_ijk[3 * e + 1], C.cell_ijk[3 * e + 2])] = e;
  const int64_t F3 = (int64_t)F.P * F.P * F.P, C3 = (int64_t)C.P * C.P * C.P, NEc = C.N + C.Nh;
  std::vector<int32_t> cf(F.n_cells * F3, -1), cc(F.n_cells * C3, -1);
  std::vector<char> taken(F.N, 0);
  for (int64_t e = 0; e < F.n_cells; ++e) {
    auto it = leaves.find(leaf_key(F.cell_level[e], F.cell_ijk[3 * e], F.cell_ijk[3 * e + 1], F.cell_ijk[3 * e + 2]));
    if (it == leaves.end()) return;   // other leaves
    for (int64_t t = 0; t < F3; ++t) {
      const int32_t nd = F.cell_nodes[e * F3 + t];
      if (nd < F.N && !taken[nd]) {
        taken[nd] = 1;
        cf[e * F3 + t] = nd;
      }
    }
    for (int64_t t = 0; t < C3; ++t) {
      const int32_t nd = C.cell_nodes[it->second * C3 + t];
      if (nd < NEc) cc[e * C3 + t] = nd;
    }
  }
  for (char t : taken)
    if (!t) return;
  lf.cell_pf = F.P;
  lf.cell_pc = C.P;
  lf.cell_f.swap(cf);
  lf.cell_c.swap(cc);
  lc.h_ptr.assign(C.Nh + 1, 0);
  for (int64_t h = 0; h < C.Nh; ++h) {
    for (int64_t t = C.hang_ptr[h]; t < C.hang_ptr[h + 1]; ++t)
      if (C.hang_col[t] < C.N) {
        lc.h_col.push_back((int32_t)C.hang_col[t]);
        lc.h_w.push_back(C.hang_w[t]);
      }
    lc.h_ptr[h + 1] = (int32_t)lc.h_col.size();
  }
}

// L <- P^T A P, A and the prolongation P from level F: row by row A P (its
// entries in order of first appearance), then each coarse row from the fine
// rows it gathers.  Entries at the rounding level of the product are dropped
// (by a symmetric test, so L stays symmetric).
void galerkin(const MgLevel& F, int64_t Nc, MgLevel& L) {
  std::vector<int32_t> ap_ptr(F.N + 1, 0), ap_col, at(Nc, -1);
  std::vector<double> ap_val;
  for (int64_t i = 0; i < F.N; ++i) {
    const int32_t beg = (int32_t)ap_col.size();
    for (int32_t t = F.k_ptr[i]; t < F.k_ptr[i + 1]; ++t) {
      const int32_t k = F.k_col[t];
      for (int32_t u = F.p_ptr[k]; u < F.p_ptr[k + 1]; ++u) {
        const int32_t c = F.p_col[u];
        const double v = F.k_val[t] * F.p_val[u];
        if (at[c] < beg) {
          at[c] = (int32_t)ap_col.size();
          ap_col.push_back(c);
          ap_val.push_back(v);
        } else {
          ap_val[at[c]] += v;
        }
      }
    }
    if (ap_col.size() >= (size_t)INT32_MAX) throw std::runtime_error("multigrid: coarse operator too large");
    ap_ptr[i + 1] = (int32_t)ap_col.size();
  }
  std::fill(at.begin(), at.end(), -1);
  L.N = Nc;
  L.k_ptr.assign(Nc + 1, 0);
  L.k_col.clear();
  L.k_val.clear();
  L.dinv.assign(Nc, 0.0);
  std::vector<double> diag(Nc, 0.0);
  std::vector<std::vector<std::pair<int32_t, double>>> rows(Nc);
  for (int64_t r = 0; r < Nc; ++r) {
    auto& row = rows[r];
    for (int32_t t = F.r_ptr[r]; t < F.r_ptr[r + 1]; ++t) {
      const int32_t i = F.r_col[t];
      for (int32_t u = ap_ptr[i]; u < ap_ptr[i + 1]; ++u) {
        const int32_t c = ap_col[u];
        const double v = F.r_val[t] * ap_val[u];
        if (at[c] < 0) {
          at[c] = (int32_t)row.size();
          row.push_back({c, v});
        } else {
          row[at[c]].second += v;
        }
      }
    }
    for (const auto& e : row) at[e.first] = -1;
    std::sort(row.begin(), row.end());
    for (const auto& e : row)
      if (e.first == r) diag[r] = e.second;
  }
  for (int64_t r = 0; r < Nc; ++r) {
    for (const auto& e : rows[r])
      if (e.second * e.second > 1e-28 * diag[r] * diag[e.first]) {
        L.k_col.push_back(e.first);
        L.k_val.push_back(e.second);
      }
    if (L.k_col.size() >= (size_t)INT32_MAX) throw std::runtime_error("multigrid: coarse operator too large");
    L.k_ptr[r + 1] = (int32_t)L.k_col.size();
    L.dinv[r] = 1.0 / diag[r];
  }
}

}  // namespace

// Operators of the levels: Q2 below Q3 is rediscretised (the Galerkin product
// would carry 60 entries a row where the collocated operator carries 13), Q1
// levels are Galerkin products P^T A P: the collocated Q1 operator, with its
// lumped mass, is stiffer than the fine one on the modes the smoother leaves.
// Iterations of the CG from zero to 1e-12, Q1 straight below Q3 and collocated
// operators -> these: H2 (Q3) 20 -> 11, a Q2 mesh of 50,429 unknowns 16 -> 12, a
// Q1 mesh of 14,205 17 -> 13.
void build_multigrid(const Mesh& fine, const OpHost& fop, MgHost& mg, int max_coarse, int threads) {
  Crew crew(threads);
  mg.lv.clear();
  std::vector<Mesh> meshes;
  meshes.push_back(fine);
  MgLevel L0;
  take_operator(fop, fine.N, L0);
  mg.lv.push_back(std::move(L0));
  // coarser meshes: Q2 on the same leaves (below Q3), Q1 on them, then shallower
  // balls (a Kelly mesh: its leaves capped one level shallower at a time, so every
  // level nests in the one above), then coarser base grids
  struct Plan {
    int nc, p;
    std::vector<Ball> balls;
    int cap;  // level cap of a Kelly mesh, -1 otherwise
  };
  std::vector<Plan> plan;
  const bool kelly = !fine.kelly.nuclei.empty();
  if (fine.p == 3) plan.push_back({fine.nc, 2, fine.balls, kelly ? fine.Lmax : -1});
  if (kelly) {
    for (int cap = fine.Lmax; cap >= 0; --cap) plan.push_back({fine.nc, 1, {}, cap});
  } else {
    int maxlev = 0;
    for (const Ball& b : fine.balls) maxlev = std::max(maxlev, b.levels);
    for (int drop = 0; drop <= maxlev; ++drop) {
      std::vector<Ball> bl;
      for (Ball b : fine.balls) {
        b.levels = std::max(0, b.levels - drop);
        if (b.levels > 0) bl.push_back(b);
      }
      plan.push_back({fine.nc, 1, bl, -1});
    }
  }
  for (int nc = fine.nc; nc % 2 == 0 && (int64_t)(nc - 1) * (nc - 1) * (nc - 1) > max_coarse;) {
    nc /= 2;
    plan.push_back({nc, 1, {}, -1});
  }
  for (size_t pi = 0; pi < plan.size(); ++pi) {
    const auto& pl = plan[pi];
    Mesh C;
    bool uns = false;
    std::string err = pl.cap >= 0 ? build_mesh(fine.lo, fine.hi, pl.nc, pl.p, {}, C, uns, nullptr, pl.cap, &fine)
                                  : build_mesh(fine.lo, fine.hi, pl.nc, pl.p, pl.balls, C, uns);
    if (!err.empty()) throw std::runtime_error("multigrid coarse mesh: " + err);
    const Mesh& F = meshes.back();
    if (F.p == 1 && C.n_cells == F.n_cells && C.nc == F.nc) continue;  // same mesh as the level above
    // a level that removes less than 40 % of the unknowns costs launches without
    // coarsening much; skip it (the meshes are nested, so the next one still is)
    if (pi + 1 < plan.size() && (double)C.N > 0.6 * (double)mg.lv.back().N) continue;
    if (C.N == 0) break;
    prolongation(F, C, mg.lv.back(), crew);
    MgLevel LC;
    if (pl.p == 1) {
      galerkin(mg.lv.back(), C.N, LC);
    } else {
      OpHost HC;
      build_poisson(C, HC, crew);
      take_operator(HC, C.N, LC);
    }
    if (F.n_cells == C.n_cells && F.nc == C.nc && F.p == C.p + 1) cell_transfer(F, C, mg.lv.back(), LC);
    mg.lv.push_back(std::move(LC));
    meshes.push_back(std::move(C));
    if (mg.lv.back().N <= max_coarse) break;  // small enough for the dense solve
  }
  for (MgLevel& L : mg.lv) L.lmax = 1.05 * lambda_max(L, crew);
  // the coarsest operator as a dense row-major matrix (inverted on the device)
  const MgLevel& Lc = mg.lv.back();
  const int64_t n = Lc.N;
  mg.coarse_dense.assign(n * n, 0.0);
  for (int64_t i = 0; i < n; ++i)
    for (int32_t t = Lc.k_ptr[i]; t < Lc.k_ptr[i + 1]; ++t) mg.coarse_dense[i * n + Lc.k_col[t]] = Lc.k_val[t];
}

}  // namespace mh
