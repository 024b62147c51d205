"""CPU run of a 2D start-up with its Richardson levels side by side: bit for bit
the levels in turn (a batch of the same instance marches them so), and the
oracle's u at lengths 3 * 2^a and with a moving well."""
import numpy as np
import pytest

from oracle.periodic import PeriodicOracle
from workloads import moving_well_problem, periodic_problem_from_seed


@pytest.mark.parametrize("order, N", [(4, 3), (6, 4), (8, 6), (8, 9)])
def test_levels_match_levels_in_turn(emu, order, N):
    from emu.emu_plan import EmuBatchPlan, EmuPlan

    prob = periodic_problem_from_seed(70 + order, 2, (64, 128), 0.002 * N, N, order=order)
    one = EmuPlan(emu, prob).run(prob.u0)
    turn = EmuBatchPlan(emu, [prob]).run([prob.u0])[0]
    assert np.array_equal(one, np.asarray(turn).reshape(one.shape))


def test_levels_match_oracle(emu):
    from emu.emu_plan import EmuPlan

    for prob in (periodic_problem_from_seed(75, 2, (24, 48), 0.01, 7, order=8, A_kind="stepwise"),
                 periodic_problem_from_seed(76, 2, (16, 96), 0.01, 5, order=6),
                 moving_well_problem(c=(10.0, 5.0), M=(32, 32), T=0.01, nsteps=8)):
        u = EmuPlan(emu, prob).run(prob.u0)
        ref, _ = PeriodicOracle(prob).run()
        assert np.linalg.norm(u - ref) / np.linalg.norm(ref) < 1e-12
