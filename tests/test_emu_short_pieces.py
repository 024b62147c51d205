"""CPU runs cut into pieces of one step, which the one-launch paths pay for with
their launches' start and end: what such a piece launches, and that it leaves
the run as the whole run has it."""
import ctypes as C

import numpy as np
import pytest

from workloads import periodic_problem_from_seed


def _state(plan, M):
    out = np.zeros(M, dtype=np.complex128)
    plan.call("tdse_get_state", C.c_void_p(out.ctypes.data), 1)
    return out


@pytest.mark.parametrize("M, order", [(32, 8), (48, 4)])
def test_persistent_pieces_mark_the_exchange_buffers_once(emu, M, order):
    from emu.emu_plan import EmuPlan

    launches = C.c_int.in_dll(emu, "emu_launches")
    prob = periodic_problem_from_seed(140 + M, 2, (M, M), 0.02, order + 12, order=order)
    plan = EmuPlan(emu, prob)
    full = plan.run(prob.u0)
    for again in range(2):
        plan.set_state(prob.u0)
        plan.step(order)
        for k in (1, 1, 3, 1):
            before = launches.value
            plan.step(k)
            assert launches.value - before == 1
        plan.query(29)                 # the residual takes the buffers for itself
        before = launches.value
        plan.step(1)
        assert launches.value - before == 2
        plan.step(5)
        assert np.array_equal(_state(plan, prob.M), full)
