"""CPU runs of the free-space line kernels for every number of grid points a
thread can hold (M <= nu/8, <= nu/2, more), at the edges of those ranges, in
both thread layouts and with direct sums and the interpolant, against the
oracle."""
import numpy as np
import pytest

from oracle.freespace import FreeSpaceOracle
from workloads import free_problem_from_seed

CASES = [
    ((32,), (256,), 8, 10, 0), ((34,), (256,), 8, 9, 0), ((128,), (256,), 4, 6, 0), ((130,), (256,), 2, 4, 0),
    ((200,), (256,), 2, 4, 20), ((32,), (256,), 4, 5, 20), ((100,), (512,), 4, 5, 20), ((256,), (2048,), 2, 3, 0),
    ((16, 128), (256, 1024), 2, 2, 0), ((40, 130), (256, 1024), 2, 2, 20), ((140, 24), (256, 256), 2, 2, 0),
]


@pytest.mark.parametrize("M, nu, order, N, cheb", CASES,
                         ids=["x".join(map(str, c[0])) + f"-nu{c[1][-1]}-c{c[4]}" for c in CASES])
def test_points_per_thread(emu, M, nu, order, N, cheb):
    from emu.emu_plan import EmuPlan

    prob = free_problem_from_seed(90 + M[0], len(M), M, 1e-3 * N, N, order=order, nu=nu, eps=1e-8, q=8)
    prob.cheb = cheb
    u = EmuPlan(emu, prob).run(prob.u0)
    ref = FreeSpaceOracle(prob).run()[0]
    assert np.linalg.norm(u - ref) <= 1e-11 * np.linalg.norm(ref)
