"""Launches of many lanes, where a row or node is taken by fewer lane groups
(batches of equal small meshes), and the complex-scaled orbital rows at every
lane width.  Bars as in test_gpu_orbital_counts: 1e-10 against the oracle."""
import copy

import numpy as np
import pytest

from synth import broad_orbitals
from tests.lib_cases import max_rel_cols, poisson_solver, rel_err_cols
from tests.test_gpu_orbital_counts import dev, frozen, orbitals, pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gauge", ["length", "velocity"])
@pytest.mark.parametrize("n,copies", [(1, 1), (2, 1), (4, 1), (5, 1), (8, 1), (1, 3), (2, 20), (4, 39), (5, 20), (8, 20)])
def test_scaled_orbital_rows(n, copies, gauge):
    """G v under complex scaling, eight or four lane groups a node (one instance) and
    four, two or one (3 to 39 instances of 6,770 nodes), v reaching into the scaled
    cells."""
    import paper_2301_02387_amd as mh
    import torch
    from oracle.ecs import ECS
    from oracle.fem import Operators
    P = copy.copy(pair("ecs_q3"))
    w = P.w
    e = w["ecs"]
    kw = dict(gauge=gauge, ecs=(e["theta"], e["inner"]), polarization=w["polarization"])
    args = (n, (n + 1) // 2, n // 2)
    if copies == 1:
        op = mh.Operator(P.mesh, w["nuclei"], *args, **kw)
    else:
        op = mh.Operator.batch([P.mesh] * copies, [w["nuclei"]] * copies, *args, **kw)
    ope = Operators(P.om, w["nuclei"], pol=w["polarization"], gauge=gauge, ecs=ECS(e["theta"], e["inner"]))
    _, fr = frozen(P, op, n, 190 + n, E=0.27, copies=copies, one_body=ope)
    xyz = P.om.xyz[P.om.dof_nodes]
    v = broad_orbitals(xyz, n, 200 + n, float(min(e["inner"])), n_gauss=n + 4)
    out = torch.zeros((P.NE * copies, n), dtype=torch.complex128, device="cuda")
    op.rhs_apply(dev(np.concatenate([P.to_lib_orb(v)] * copies)), out)
    torch.cuda.synchronize()
    ref = fr.G(v)
    for part in np.split(out.cpu().numpy(), copies):
        got = P.from_lib_dof(part)
        assert rel_err_cols(got, ref) < 1e-10 and max_rel_cols(got, ref) < 1e-10


@pytest.mark.parametrize("gauge", ["length", "velocity"])
@pytest.mark.parametrize("n,copies", [(1, 2), (1, 3), (2, 21), (2, 22), (3, 5), (3, 6), (7, 2), (7, 3)])
def test_orbital_rows_bound(n, copies, gauge):
    """G v on both sides of the lane counts (2^14 lanes of one orbital, 2^18 of two, else 2^17)
    where a node is taken by fewer lane groups."""
    import paper_2301_02387_amd as mh
    import torch
    from oracle.fem import Operators
    P = copy.copy(pair("tiny_q3"))
    op = mh.Operator.batch([P.mesh] * copies, [P.w["nuclei"]] * copies, n, (n + 1) // 2, n // 2, gauge=gauge)
    ops = P.ops if gauge == "length" else Operators(P.om, P.w["nuclei"], gauge="velocity")
    _, fr = frozen(P, op, n, 220 + n, E=0.31, copies=copies, one_body=ops)
    v = orbitals(P, n, 230 + n)
    out = torch.zeros((P.NE * copies, n), dtype=torch.complex128, device="cuda")
    op.rhs_apply(dev(np.concatenate([P.to_lib_orb(v)] * copies)), out)
    torch.cuda.synchronize()
    ref = fr.G(v)
    for part in np.split(out.cpu().numpy(), copies):
        got = P.from_lib_dof(part)
        assert rel_err_cols(got, ref) < 1e-10 and max_rel_cols(got, ref) < 1e-10


@pytest.mark.parametrize("n,copies", [(1, 910), (2, 228), (3, 58)])
def test_level_passes_one_group(n, copies):
    """Coarse-level passes below 16 columns with one lane group a row (a Q2 level of
    1,153 unknowns an instance): potentials of every instance, and the iterations,
    as in test_multigrid_degree_levels."""
    import paper_2301_02387_amd as mh
    import torch
    P = pair("tiny_q3")
    op = mh.Operator.batch([P.mesh] * copies, [P.w["nuclei"]] * copies, n, (n + 1) // 2, n // 2, poisson_rtol=1e-13,
                           poisson_maxit=20000)
    op.tune(1, 21, 8192)
    c = orbitals(P, n, 210 + n)
    W = torch.zeros((P.NF * copies, n * n), dtype=torch.float64, device="cuda")
    it, rc = op.poisson_pairs(dev(np.concatenate([P.to_lib_orb(c)] * copies)), W)
    torch.cuda.synchronize()
    assert rc == 0 and it <= 26
    ref = poisson_solver(P.ops).pair_potentials(c)
    parts = W.view(copies, P.NF, n * n)
    # every instance against the first by itself on the device (1e-11: FP64 atomic
    # order), the first and the last against the oracle
    assert float((parts - parts[:1]).abs().max() / parts[0].abs().max()) <= 1e-11
    for i in (0, copies - 1):
        got = P.W_from_lib(parts[i].cpu().numpy(), n)
        for k in ref:
            assert np.abs(got[k] - ref[k]).max() <= 1e-10 * np.abs(ref[k]).max()
