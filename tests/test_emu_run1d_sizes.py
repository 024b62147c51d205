"""CPU run of the one-workgroup 1D path at the lengths where its layouts differ:
3 * 2^a (a third of the threads has no physical points) with held and with
LDS twiddles, and the longest line; against the oracle (1e-12, as the path's
other lengths), and in pieces, bit for bit."""
import ctypes as C

import numpy as np
import pytest

from oracle.periodic import PeriodicOracle
from workloads import periodic_problem_from_seed


@pytest.mark.parametrize("M,order,A_kind", [(24, 8, "pulse_sin2"), (96, 4, "pulse_sin2"), (384, 8, "none"),
                                            (768, 8, "pulse_sin2"), (2048, 6, "stepwise")])
def test_run1d_lengths(emu, M, order, A_kind):
    from emu.emu_plan import EmuPlan

    prob = periodic_problem_from_seed(40 + M, 1, (M,), 0.04, 9 + order, order=order, A_kind=A_kind)
    plan = EmuPlan(emu, prob)
    plan.call("tdse_profile", 1)
    full = plan.run(prob.u0)
    assert plan.query(25) == 1.0 and plan.query(11) == 0.0
    ref, _ = PeriodicOracle(prob).run()
    assert np.linalg.norm(full - ref) / np.linalg.norm(ref) < 1e-12
    pieces = EmuPlan(emu, prob)
    pieces.set_state(prob.u0)
    for k in (order - 1, 1, 2, 7):
        pieces.step(k)
    out = np.zeros(prob.M, dtype=np.complex128)
    pieces.call("tdse_get_state", C.c_void_p(out.ctypes.data), 1)
    assert np.array_equal(out, full)
