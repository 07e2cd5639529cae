"""Pair solves under different Poisson schedules in turn on one handle (their
workspaces are shared: the Jacobi CG keeps z = D^-1 r where the right-hand side
had its boundary lift): every order against the oracle's direct solve, and the
same iteration counts as on a handle that runs one schedule alone.  Bars as in
test_gpu_orbital_counts."""
import numpy as np
import pytest

from tests.lib_cases import poisson_solver
from tests.test_gpu_orbital_counts import dev, orbitals, pair

pytestmark = pytest.mark.gpu


def handle(P, n, copies):
    import paper_2301_02387_amd as mh
    args = (n, (n + 1) // 2, n // 2)
    kw = dict(poisson_rtol=1e-13, poisson_maxit=20000)
    if copies == 1:
        return mh.Operator(P.mesh, P.w["nuclei"], *args, **kw)
    return mh.Operator.batch([P.mesh] * copies, [P.w["nuclei"]] * copies, *args, **kw)


@pytest.mark.parametrize("copies", [1, 2])
@pytest.mark.parametrize("n,order", [(1, (37, 5, 4)), (3, (5, 37, 21, 36)), (5, (21, 0, 37)), (6, (13, 45, 2, 34)),
                                     (8, (37, 21, 130, 5))])
def test_schedules_in_turn(n, order, copies):
    """Rows by waves and not, the sliced-ELL copy, column blocks, and multigrid
    solves between them; the second solve of each from a warm start."""
    import torch
    P = pair("tiny_q3")
    c = orbitals(P, n, 160 + n)
    x = dev(np.concatenate([P.to_lib_orb(c)] * copies))
    ref = poisson_solver(P.ops).pair_potentials(c)
    op = handle(P, n, copies)
    for sched in order:
        its = []
        for o in (op, handle(P, n, copies)):
            o.tune(1, sched, 8192)
            W = torch.zeros((P.NF * copies, n * n), dtype=torch.float64, device="cuda")
            it, rc = o.poisson_pairs(x, W)
            torch.cuda.synchronize()
            assert rc == 0
            its.append(it)
            W *= 1.0 + 1e-5
            it, rc = o.poisson_pairs(x, W, warm=True)
            torch.cuda.synchronize()
            assert rc == 0
            its.append(it)
            for part in np.split(W.cpu().numpy(), copies):
                got = P.W_from_lib(part, n)
                for k in ref:
                    assert np.abs(got[k] - ref[k]).max() <= 1e-10 * np.abs(ref[k]).max(), (sched, k)
        # sums in another order only: at most one check interval of the Jacobi CG apart
        assert abs(its[0] - its[2]) <= 8 and abs(its[1] - its[3]) <= 8
