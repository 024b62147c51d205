"""CPU run of the whole-run graph replay through the emulation harness (a
captured stream's launches and copies are kept and run again): plans whose
persistent launch does not fit the device, and the guard's check after a
replay."""
import ctypes as C

import numpy as np
import pytest

from workloads import periodic_problem_from_seed


def _graph_plan(emu, prob):
    from emu.emu_plan import EmuPlan

    plan = EmuPlan(emu, prob)
    plan._stream = C.create_string_buffer(8)   # graph replay needs a stream that is not the default one
    plan.call("tdse_bind", C.c_void_p(plan.ws.ctypes.data), plan.ws.size, C.cast(plan._stream, C.c_void_p))
    plan.call("tdse_graph", 1)
    return plan


@pytest.fixture
def coop_blocks(emu):
    knob = C.c_int.in_dll(emu, "emu_coop_blocks")
    yield knob
    knob.value = 1


@pytest.mark.parametrize("M", [32, 48])
def test_replay_after_the_persistent_launch_did_not_fit(emu, coop_blocks, M):
    prob = periodic_problem_from_seed(90 + M, 2, (M, M), 0.02, 12, order=4)
    plan = _graph_plan(emu, prob)
    plan.call("tdse_configure", 0, 0)
    passes = plan.run(prob.u0)
    plan.call("tdse_configure", 0, 1)
    coop_blocks.value = 0
    for rep in range(3):
        assert np.array_equal(plan.run(prob.u0), passes), rep
    assert plan.query(28) == 0.0


@pytest.mark.parametrize("M", [(32,), (24, 32)])
def test_guard_after_a_replay_scans_the_final_state(emu, M):
    """An odd number of start-up steps leaves u in the second physical buffer."""
    prob = periodic_problem_from_seed(95, len(M), M, 0.5, 5, order=2)
    prob.n_start = 3
    plan = _graph_plan(emu, prob)
    plan.call("tdse_configure", 1, 1)
    for rep in range(3):
        u0 = (1.0 + rep) * np.asarray(prob.u0)
        u = plan.run(u0)
        assert abs(plan.query(30) - np.linalg.norm(u)) <= 1e-12 * np.linalg.norm(u), rep
