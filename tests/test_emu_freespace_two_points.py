"""CPU runs of the free-space line kernels with two grid points per thread
(nu/8 < M <= nu/4), at the edges of that range, in every line kernel and with
direct sums and the interpolant, against the oracle."""
import numpy as np
import pytest

from oracle.freespace import FreeSpaceOracle
from workloads import free_problem_from_seed

CASES = [
    ((38,), (256,), 4, 6, 0), ((64,), (256,), 8, 9, 0), ((66,), (256,), 2, 4, 20), ((256,), (1024,), 2, 3, 0),
    ((40, 150), (256, 1024), 2, 2, 0), ((150, 40), (1024, 256), 2, 2, 20),
]


@pytest.mark.parametrize("M, nu, order, N, cheb", CASES,
                         ids=["x".join(map(str, c[0])) + f"-nu{c[1][-1]}-c{c[4]}" for c in CASES])
def test_two_points_per_thread(emu, M, nu, order, N, cheb):
    from emu.emu_plan import EmuPlan

    prob = free_problem_from_seed(120 + M[0], len(M), M, 1e-3 * N, N, order=order, nu=nu, eps=1e-8, q=8)
    prob.cheb = cheb
    u = EmuPlan(emu, prob).run(prob.u0)
    ref = FreeSpaceOracle(prob).run()[0]
    assert np.linalg.norm(u - ref) <= 1e-11 * np.linalg.norm(ref)
