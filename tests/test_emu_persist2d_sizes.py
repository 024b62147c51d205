"""CPU run of the persistent 2D Adams steps at lengths 3 * 2^a (four and three
elements per thread in the two layouts) through the emulation harness: against the oracle and the
two-pass path, with and without a field along axis 1."""
import numpy as np
import pytest

from oracle.periodic import PeriodicOracle
from workloads import periodic_problem_from_seed


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("M, order, dir2", [(48, 8, True), (96, 4, False)])
def test_persistent_three_smooth_sizes(emu, M, order, dir2):
    from emu.emu_plan import EmuPlan

    prob = periodic_problem_from_seed(47 + M, 2, (M, M), 0.03, 9, order=order)
    if dir2:
        prob.A_params = prob.A_params[:3] + (0.6, -0.8)
    plan = EmuPlan(emu, prob)
    assert plan.query(28) == 2.0
    u = plan.run(prob.u0)
    assert _rel(u, PeriodicOracle(prob).run()[0]) < 1e-12
    plan.call("tdse_configure", 0, 0)
    assert _rel(u, plan.run(prob.u0)) < 1e-13
