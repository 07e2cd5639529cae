"""The timing hook records every Poisson operator launch of the CG: one per
iteration and, where the solve starts from a given potential, the pass that
forms its first residual."""
import pytest

from tests.test_gpu_orbital_counts import dev, operator, orbitals, pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sched", [5, 21, 85, 23])
@pytest.mark.parametrize("n", [2, 8])
def test_poisson_launches_recorded(n, sched):
    """Jacobi and multigrid, the finest level in double and in float, column
    blocks (8 orbitals, schedule bit 1)."""
    import torch
    P = pair("tiny_q2")
    op = operator(P, n)
    op.tune(1, sched, 8192)
    c = dev(P.to_lib_orb(orbitals(P, n, 30 + n)))
    W = torch.zeros((P.NF, n * n), dtype=torch.float64, device="cuda")
    op.kernel_timing(1, True)
    it, rc = op.poisson_pairs(c, W)
    avg, count = op.kernel_timing(1, True)
    assert rc == 0 and count == it and avg > 0.0
    W *= 1.0 + 1e-6
    it, rc = op.poisson_pairs(c, W, warm=True)
    avg, count = op.kernel_timing(1, False)
    assert rc == 0 and it > 0 and count == it + 1 and avg > 0.0
