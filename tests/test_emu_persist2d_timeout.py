"""CPU run of a persistent 2D launch whose exchanges time out (the emulated
build's poll limit set to none from the host): the plan reports it, takes no further step
and hands out no state, and marches again after a new one; and a step makes no
call that waits for the stream."""
import ctypes as C

import numpy as np
import pytest

from workloads import periodic_problem_from_seed

EDEVICE, ESTATE = -4, -6


@pytest.fixture
def spin_limit(emu):
    knob = C.c_int.in_dll(emu, "emu_spin_limit")
    usual = knob.value
    yield knob
    knob.value = usual


def _plan(emu, M, nsteps=12):
    from emu.emu_plan import EmuPlan

    prob = periodic_problem_from_seed(50 + M, 2, (M, M), 0.02, nsteps, order=4)
    plan = EmuPlan(emu, prob)
    assert plan.query(28) == 2.0
    return prob, plan


@pytest.mark.parametrize("M", [32, 48])
def test_a_timed_out_run_is_reported_and_not_continued(emu, spin_limit, M):
    prob, plan = _plan(emu, M)
    ref = plan.run(prob.u0)
    assert np.isfinite(ref).all()
    plan.set_state(prob.u0)
    spin_limit.value = 0
    assert emu.tdse_step(plan.h, 8) == EDEVICE
    assert b"timed out" in emu.tdse_last_error()
    spin_limit.value = 1000000
    out = np.zeros(prob.M, dtype=np.complex128)
    assert emu.tdse_step(plan.h, 1) == ESTATE
    assert emu.tdse_get_state(plan.h, C.c_void_p(out.ctypes.data), 1) == ESTATE
    assert np.array_equal(plan.run(prob.u0), ref)
    spin_limit.value = 0
    assert emu.tdse_run(plan.h, C.c_void_p(np.asarray(prob.u0).ctypes.data), C.c_void_p(out.ctypes.data), 1) == EDEVICE


@pytest.mark.parametrize("M", [32, 48])
def test_steps_do_not_wait_for_the_stream(emu, M):
    waits = C.c_int.in_dll(emu, "emu_stream_waits")
    prob, plan = _plan(emu, M)
    plan.set_state(prob.u0)
    before = waits.value
    for k in (2, 5, 1, 4):
        plan.step(k)
    assert waits.value == before
    plan.set_state(prob.u0)            # the next run waits for the last one's launch
    assert waits.value == before + 1
    plan.run(prob.u0)                  # (no launch under way) and a run for its own
    assert waits.value == before + 2
    plan.set_state(prob.u0)
    assert waits.value == before + 2
