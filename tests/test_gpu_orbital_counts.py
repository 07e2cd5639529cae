"""Kernels whose tiling follows the orbital count (1 to 8 orbitals: 1 to 64
real pair columns), against the CPU oracle on small meshes.

Bars as in test_gpu_parity: potentials <= 1e-10 in the m-weighted norm and
element-wise (CG to a relative residual of 1e-13 against a direct solve)."""
import numpy as np
import pytest

from synth import random_orbitals
from tests.lib_cases import Pair, poisson_solver

pytestmark = pytest.mark.gpu

_PAIRS = {}


def pair(name):
    if name not in _PAIRS:
        _PAIRS[name] = Pair(name, with_op=False)
    return _PAIRS[name]


def operator(P, n, **kw):
    import paper_2301_02387_amd as mh
    return mh.Operator(P.mesh, P.w["nuclei"], n, (n + 1) // 2, n // 2, poisson_rtol=1e-13, poisson_maxit=20000, **kw)


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def orbitals(P, n, seed):
    from oracle.mctdhf import orthonormalize
    return orthonormalize(P.ops, random_orbitals(P.om.xyz[P.om.dof_nodes], n, seed, n_gauss=10, spread=1.5))


@pytest.mark.parametrize("sched", [21, 85])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("name", ["tiny_q3", "tiny_q2", "uniform_q2"])
def test_multigrid_degree_levels(name, n, sched):
    """Hierarchies whose first levels lie on the same leaves (Q3 - Q2 - Q1, with
    and without hanging nodes): transfers cell by cell, lane groups of the
    coarse passes at every column count, the finest corrections in double and in
    float.  A wrong transfer or smoothing step costs iterations, not accuracy, so
    those are held as well: the cycle gains a digit an iteration, 13 are asked
    for, twice as many are allowed."""
    import torch
    P = pair(name)
    op = operator(P, n)
    op.tune(1, sched, 8192)
    c = orbitals(P, n, 60 + n)
    W = torch.zeros((P.NF, n * n), dtype=torch.float64, device="cuda")
    it, rc = op.poisson_pairs(dev(P.to_lib_orb(c)), W)
    torch.cuda.synchronize()
    assert rc == 0 and it <= 26
    got, ref = P.W_from_lib(W.cpu().numpy(), n), poisson_solver(P.ops).pair_potentials(c)
    m = P.ops.m
    for k in ref:
        scale = np.sqrt(np.sum(m * np.abs(ref[k]) ** 2))
        assert np.sqrt(np.sum(m * np.abs(got[k] - ref[k]) ** 2)) <= 1e-10 * scale
        assert np.abs(got[k] - ref[k]).max() <= 1e-10 * np.abs(ref[k]).max()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("name", ["uniform_q1_odd", "tiny_q1"])
def test_multigrid_column_tiles(name, n):
    """Multigrid-preconditioned pair solves at every column count: the dense
    coarsest solve alone (odd grid, one level: 64 unknowns, whole row tiles)
    and below smoothed levels (ragged row tiles)."""
    import torch
    P = pair(name)
    op = operator(P, n)
    op.tune(1, 21, 8192)
    c = orbitals(P, n, 40 + n)
    W = torch.zeros((P.NF, n * n), dtype=torch.float64, device="cuda")
    it, rc = op.poisson_pairs(dev(P.to_lib_orb(c)), W)
    torch.cuda.synchronize()
    assert rc == 0
    got, ref = P.W_from_lib(W.cpu().numpy(), n), poisson_solver(P.ops).pair_potentials(c)
    m = P.ops.m
    for k in ref:
        scale = np.sqrt(np.sum(m * np.abs(ref[k]) ** 2))
        assert np.sqrt(np.sum(m * np.abs(got[k] - ref[k]) ** 2)) <= 1e-10 * scale
        assert np.abs(got[k] - ref[k]).max() <= 1e-10 * np.abs(ref[k]).max()


def test_multigrid_cells_wide():
    """41 equal instances at 8 orbitals (535,000 cell columns): the cell-by-cell
    prolongation with a whole cell per thread; each against the oracle."""
    import paper_2301_02387_amd as mh
    import torch
    P, n, copies = pair("tiny_q3"), 8, 41
    op = mh.Operator.batch([P.mesh] * copies, [P.w["nuclei"]] * copies, n, 4, 4, poisson_rtol=1e-13,
                           poisson_maxit=20000)
    op.tune(1, 21, 8192)
    c = orbitals(P, n, 75)
    W = torch.zeros((P.NF * copies, n * n), dtype=torch.float64, device="cuda")
    it, rc = op.poisson_pairs(dev(np.concatenate([P.to_lib_orb(c)] * copies)), W)
    torch.cuda.synchronize()
    assert rc == 0 and it <= 26
    ref = poisson_solver(P.ops).pair_potentials(c)
    for part in np.split(W.cpu().numpy(), copies):
        got = P.W_from_lib(part, n)
        for k in ref:
            assert np.abs(got[k] - ref[k]).max() <= 1e-10 * np.abs(ref[k]).max()


def frozen(P, op, n, seed, E=0.013, copies=1, one_body=None):
    """Oracle frozen operator and the library (a handle of `copies` equal instances) frozen on the same inputs."""
    from oracle.ci import CISpace
    from oracle.mctdhf import Frozen
    from synth import random_ci
    c = orbitals(P, n, seed)
    cs = CISpace(n, (n + 1) // 2, n // 2)
    gam, Gam = cs.rdms(random_ci(cs.dim, seed + 1))
    W = poisson_solver(P.ops).pair_potentials(c)
    rep = lambda a: dev(np.concatenate([a] * copies))  # noqa: E731
    op.freeze(rep(P.to_lib_orb(c)), rep(gam), rep(Gam), E, rep(P.W_to_lib(W, n)))
    return c, Frozen(one_body or P.ops, c, gam, Gam, E, W)


def check_arnoldi(P, op, c, fr, tau, m, copies=1):
    import torch
    from oracle.mctdhf import arnoldi_step
    from tests.lib_cases import rel_err_cols, max_rel_cols
    x = dev(np.concatenate([P.to_lib_orb(c)] * copies))
    err, m_used = op.arnoldi_step(x, tau, m)
    torch.cuda.synchronize()
    ref, err_ref, m_ref, H = arnoldi_step(P.ops, fr.G, c, tau, m)
    assert m_used == m_ref
    for part in np.split(x.cpu().numpy(), copies):
        got = P.from_lib_dof(part)
        assert rel_err_cols(got, ref) < 1e-10
        assert max_rel_cols(got, ref) < 1e-10
    assert abs(err - err_ref) <= 1e-6 * err_ref + 1e-14
    return H


@pytest.mark.parametrize("copies", [1, 2])
@pytest.mark.parametrize("n,m", [(1, 4), (2, 5), (3, 8), (4, 9), (5, 13), (6, 12), (7, 14), (8, 12)])
def test_arnoldi_vectors(n, m, copies):
    """Krylov vectors of every orbital count and the register tiles' edges (4,
    8, 13 basis vectors), with the partial sums folded by the next launch (one
    instance) and by a launch of their own (a batch)."""
    import paper_2301_02387_amd as mh
    P = pair("tiny_q1")
    if copies == 1:
        op = operator(P, n)
    else:
        op = mh.Operator.batch([P.mesh] * copies, [P.w["nuclei"]] * copies, n, (n + 1) // 2, n // 2)
    c, fr = frozen(P, op, n, 60 + n, copies=copies)
    check_arnoldi(P, op, c, fr, 0.02, m, copies)


@pytest.mark.parametrize("gauge", ["length", "velocity"])
@pytest.mark.parametrize("n,copies", [(1, 1), (2, 1), (3, 1), (4, 1), (6, 1), (8, 1), (3, 43), (4, 43), (5, 22), (8, 22)])
def test_orbital_rows(n, copies, gauge):
    """G v by rows at every lane width, with four lane groups a node (one
    instance) and with one or two (above 2^20 lanes: 22 or 43 instances)."""
    import copy
    import paper_2301_02387_amd as mh
    import torch
    from oracle.fem import Operators
    from tests.lib_cases import rel_err_cols, max_rel_cols
    P = copy.copy(pair("tiny_q3"))
    kw = dict(gauge=gauge)
    if copies == 1:
        op = mh.Operator(P.mesh, P.w["nuclei"], n, (n + 1) // 2, n // 2, **kw)
    else:
        op = mh.Operator.batch([P.mesh] * copies, [P.w["nuclei"]] * copies, n, (n + 1) // 2, n // 2, **kw)
    ops = P.ops if gauge == "length" else Operators(P.om, P.w["nuclei"], gauge="velocity")
    _, fr = frozen(P, op, n, 100 + n, E=0.31, copies=copies, one_body=ops)
    v = orbitals(P, n, 120 + n)
    out = torch.zeros((P.NE * copies, n), dtype=torch.complex128, device="cuda")
    op.rhs_apply(dev(np.concatenate([P.to_lib_orb(v)] * copies)), out)
    torch.cuda.synchronize()
    ref = fr.G(v)
    for part in np.split(out.cpu().numpy(), copies):
        got = P.from_lib_dof(part)
        assert rel_err_cols(got, ref) < 1e-10 and max_rel_cols(got, ref) < 1e-10


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8])
def test_mass_solve_in_place(n):
    """The mass solve by the dense inverse at every orbital width, into another
    array (one launch) and in place (masters gathered first): the same values,
    and M c = f."""
    import torch
    from tests.lib_cases import rel_err_cols
    P = pair("tiny_q3")
    op = operator(P, n)
    f = dev(P.to_lib_orb(orbitals(P, n, 140 + n)))
    c = torch.zeros_like(f)
    op.mass_solve(f, c)
    g = f.clone()
    op.mass_solve(g, g)
    torch.cuda.synchronize()
    assert torch.equal(c, g)
    ref = P.from_lib_dof(f.cpu().numpy()[:P.N])
    assert rel_err_cols(P.ops.M @ P.from_lib_dof(c.cpu().numpy()), ref) < 1e-10


@pytest.mark.parametrize("copies", [1, 2])
def test_arnoldi_second_pass(copies):
    """A start vector near an eigenvector of G: the first Gram-Schmidt pass
    keeps less than a tenth of G v_0, so the second one runs."""
    import paper_2301_02387_amd as mh
    P = pair("beta_one")
    nuc = P.w["nuclei"]
    op = mh.Operator(P.mesh, nuc, 1, 1, 0) if copies == 1 else mh.Operator.batch([P.mesh] * 2, [nuc] * 2, 1, 1, 0)
    _, fr = frozen(P, op, 1, 80, copies=copies)
    N = P.N
    G = np.stack([fr.G(e[:, None])[:, 0] for e in np.eye(N, dtype=complex)], axis=1)
    lam, X = np.linalg.eig(G)
    x = X[:, np.argsort(-np.abs(lam))[3]]
    rng = np.random.default_rng(5)
    x = x + 1e-3 * np.linalg.norm(x) / np.sqrt(N) * (rng.standard_normal(N) + 1j * rng.standard_normal(N))
    H = check_arnoldi(P, op, x[:, None], fr, 0.02, 6, copies)
    assert np.abs(H[1, 0]) < 0.1 * np.linalg.norm(H[:2, 0])


@pytest.mark.parametrize("n,na,nb", [(1, 1, 0), (2, 1, 1), (2, 2, 1), (3, 2, 1), (4, 3, 2), (5, 2, 3), (5, 3, 2), (6, 3, 2),
                                     (7, 4, 3), (8, 5, 5)])
@pytest.mark.parametrize("copies", [1, 2])
def test_rdms_tiles(n, na, nb, copies):
    """RDMs at every pair-tile count, in one workgroup (at most 64
    determinants) and with partial sums, ragged last chunks among them; sums of
    at most 3,136 products of amplitudes of a unit vector: 1e-13."""
    import torch
    import paper_2301_02387_amd as mh
    from oracle.ci import CISpace
    from synth import random_ci
    P = pair("uniform_q1_odd")
    op = mh.Operator.batch([P.mesh] * copies, [P.w["nuclei"]] * copies, n, na, nb)
    cs = CISpace(n, na, nb)
    C = np.stack([random_ci(cs.dim, 90 + i) for i in range(copies)])
    gam = torch.zeros((copies, n, n), dtype=torch.complex128, device="cuda")
    Gam = torch.zeros((copies, n, n, n, n), dtype=torch.complex128, device="cuda")
    op.ci_rdms(dev(C), gam, Gam)
    torch.cuda.synchronize()
    for i in range(copies):
        g_ref, G_ref = cs.rdms(C[i])
        assert np.abs(gam[i].cpu().numpy() - g_ref).max() <= 1e-13
        assert np.abs(Gam[i].cpu().numpy() - G_ref).max() <= 1e-13


@pytest.mark.parametrize("n,na,nb", [(2, 1, 1), (3, 2, 1), (4, 2, 2), (4, 3, 3), (5, 2, 2), (6, 2, 1)])
def test_ci_step_sizes(n, na, nb):
    """Two coupled steps with the CI exponential in one workgroup (up to 64
    determinants and 1,024 amplitudes: 4, 9, 36, 16 determinants) and by the
    launches beyond (100 and 90 determinants, the 12-vector space)."""
    import torch
    import paper_2301_02387_amd as mh
    from oracle.ci import CISpace
    from oracle.mctdhf import Propagator
    from synth import random_ci
    from tests.lib_cases import rel_err_cols
    P = pair("tiny_q1")
    op = mh.Operator(P.mesh, P.w["nuclei"], n, na, nb, poisson_rtol=1e-13, poisson_maxit=20000)
    op.tune(1, 53, 8192)
    cs = CISpace(n, na, nb)
    c, C = orbitals(P, n, 70 + n), random_ci(cs.dim, 71)
    pr = Propagator(P.ops, cs, poisson_solver(P.ops))
    cr, Cr = c, C
    for E in (0.01, 0.03):
        cr, Cr, _ = pr.step(cr, Cr, E, 0.02, 10)
    x, Cd = dev(P.to_lib_orb(c)), dev(C)
    W = torch.zeros((P.NF, n * n), dtype=torch.float64, device="cuda")
    op.propagate(x, Cd, W, [0.01, 0.03, 0.0], 0.02, m=10, final=False)
    torch.cuda.synchronize()
    assert np.linalg.norm(Cd.cpu().numpy().ravel() - Cr) <= 1e-8
    assert rel_err_cols(P.from_lib_dof(x.cpu().numpy()), cr) <= 1e-8
