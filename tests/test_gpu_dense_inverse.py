"""The dense inverses made on the device (Gauss-Jordan by blocks of 32 pivots):
the interface block's through the mass solve, the coarsest multigrid level's
through the preconditioned CG.

Interface block: condition number below 2, at most 1,220 unknowns, so an inverse
good to rounding leaves M c = f to about 1e-15; 1e-13 is asked for.  Coarsest
level alone (one level): the CG is exact after one iteration but for rounding,
two are allowed."""
import numpy as np
import pytest

from tests.lib_cases import rel_err_cols
from tests.test_gpu_orbital_counts import dev, operator, orbitals, pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3])
@pytest.mark.parametrize("name", ["tiny_q1", "tiny_q2", "tiny_q3", "kelly_q1", "kelly_q2", "ecs_q2"])
def test_interface_block(name, n):
    """87, 26, 459, 670, 1,220 and 90 unknowns: less than a block of pivots, ragged
    last blocks of pivots and of rows."""
    import torch
    P = pair(name)
    op = operator(P, n)
    f = dev(P.to_lib_orb(orbitals(P, n, 170 + n)))
    c = torch.zeros_like(f)
    op.mass_solve(f, c)
    torch.cuda.synchronize()
    ref = P.from_lib_dof(f.cpu().numpy()[:P.N])
    assert rel_err_cols(P.ops.M @ P.from_lib_dof(c.cpu().numpy()), ref) < 1e-13


@pytest.mark.parametrize("n_coarse", [2, 3, 4, 5, 9])
def test_coarsest_level_alone(n_coarse):
    """An unrefined Q1 grid is one level: 1, 8, 27, 64 and 512 unknowns (less than
    a block of pivots, two whole blocks, several tiles)."""
    import torch
    import paper_2301_02387_amd as mh
    w = dict(name="uniform", lo=-4.0, hi=4.0, n_coarse=n_coarse, p=1, balls=[], nuclei=[(1.0, (0.3, -0.2, 0.1))],
             n_orb=1, n_alpha=1, n_beta=0)
    mesh = mh.Mesh.from_workload(w)
    op = mh.Operator(mesh, w["nuclei"], 1, 1, 0, poisson_rtol=1e-12, poisson_maxit=50)
    op.tune(1, 21, 8192)
    rng = np.random.default_rng(n_coarse)
    x = rng.standard_normal((op.n_ext, 1)) + 1j * rng.standard_normal((op.n_ext, 1))
    W = torch.zeros((op.n_full, 1), dtype=torch.float64, device="cuda")
    it, rc = op.poisson_pairs(dev(x), W)
    torch.cuda.synchronize()
    assert op.n_dof == (n_coarse - 1) ** 3
    assert rc == 0 and it <= 2


@pytest.mark.parametrize("n", [3, 4, 5, 8])
def test_load_vector_gathered_or_laid_out(n):
    """1,220 masters on both sides of 5,400 values: the mass solve into another array
    (masters' rows gathered by every workgroup, or laid out first) and in place."""
    import torch
    P = pair("kelly_q2")
    op = operator(P, n)
    f = dev(P.to_lib_orb(orbitals(P, n, 180 + n)))
    c, g = torch.zeros_like(f), f.clone()
    op.mass_solve(f, c)
    op.mass_solve(g, g)
    torch.cuda.synchronize()
    assert torch.equal(c, g)
    ref = P.from_lib_dof(f.cpu().numpy()[:P.N])
    assert rel_err_cols(P.ops.M @ P.from_lib_dof(c.cpu().numpy()), ref) < 1e-13
