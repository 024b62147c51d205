"""CPU runs of the one-workgroup 1D free-space Adams steps through the
emulation harness: against the oracle over orders, interpolant and several
launches per run, in pieces, and against the general passes (a profiled run
takes those), with the evaluation outside [-1, 1] that reads the final modes."""
import ctypes as C

import numpy as np
import pytest

from oracle.freespace import FreeSpaceOracle
from workloads import free_problem_from_seed

CASES = [((32,), (256,), 8, 30, 0), ((100,), (512,), 4, 12, 0), ((24,), (256,), 2, 9, 0), ((140,), (256,), 6, 10, 0),
         ((40,), (512,), 8, 12, 20), ((16,), (256,), 2, 150, 0)]


def _problem(M, nu, order, N, cheb):
    prob = free_problem_from_seed(60 + M[0], 1, M, 1e-3 * N, N, order=order, nu=nu, eps=1e-8, q=8)
    prob.cheb = cheb
    return prob


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("M, nu, order, N, cheb", CASES, ids=[f"{c[0][0]}-nu{c[1][0]}-o{c[2]}-c{c[4]}" for c in CASES])
def test_run_matches_oracle_and_passes(emu, M, nu, order, N, cheb):
    from emu.emu_plan import EmuPlan

    prob = _problem(M, nu, order, N, cheb)
    plan = EmuPlan(emu, prob)
    u = plan.run(prob.u0)
    assert _rel(u, FreeSpaceOracle(prob).run()[0]) <= 1e-11
    plan.call("tdse_profile", 1)
    two = plan.run(prob.u0)
    assert plan.query(11) > 0        # timed row passes: the general path
    assert 0.0 < _rel(u, two) <= 1e-12 or np.array_equal(u, two)


def test_run_in_pieces(emu):
    from emu.emu_plan import EmuPlan

    prob = _problem(*CASES[0])
    plan = EmuPlan(emu, prob)
    full = plan.run(prob.u0)
    plan.set_state(prob.u0)
    out = np.zeros(prob.M, dtype=np.complex128)
    for k in (3, 3, 1, 5, 10, 8):    # start-up, to the Adams start, then pieces
        plan.step(k)
        plan.call("tdse_get_state", C.c_void_p(out.ctypes.data), 1)
    assert _rel(out, full) <= 1e-13
