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
