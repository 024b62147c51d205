"""Which path a run takes, shown by what it launches on the CPU build: the
one-workgroup 1D free-space run and the start-up levels side by side, each
against the general passes of the same problem (not bit for bit theirs in
free space, so the two are different code)."""
import ctypes as C

import numpy as np
import pytest

from workloads import free_problem_from_seed, periodic_problem_from_seed

Q_PATH, Q_LEVELS = 28, 31


def _launches(emu, call):
    n = C.c_int.in_dll(emu, "emu_launches")
    before = n.value
    call()
    return n.value - before


@pytest.mark.parametrize("M, nu, order, cheb", [(32, 256, 8, 0), (100, 256, 4, 0), (140, 256, 6, 0), (40, 512, 8, 20)])
def test_free_1d_run_is_one_launch(emu, M, nu, order, cheb):
    from emu.emu_plan import EmuPlan

    prob = free_problem_from_seed(180 + M, 1, (M,), 0.01, order + 20, order=order, nu=(nu,), eps=1e-8, q=8)
    prob.cheb = cheb
    plan = EmuPlan(emu, prob)
    assert plan.query(Q_PATH) == 3.0
    plan.set_state(prob.u0)
    plan.step(order)
    assert _launches(emu, lambda: plan.step(12)) == 2      # the factors, then every step
    assert plan.query(Q_PATH) == 3.0
    u = plan.run(prob.u0)
    plan.call("tdse_profile", 1)
    plan.set_state(prob.u0)
    assert plan.query(Q_PATH) == 0.0
    plan.step(order)
    assert _launches(emu, lambda: plan.step(12)) == 24     # two passes per step
    two = plan.run(prob.u0)
    assert not np.array_equal(u, two)
    assert np.linalg.norm(u - two) <= 1e-12 * np.linalg.norm(two)


@pytest.mark.parametrize("M, order, precision, levels", [((32, 64), 8, "fp64", 4), ((24, 48), 4, "fp64", 2),
                                                         ((32, 64), 8, "fp32split", 1), ((64,), 8, "fp64", 1)])
def test_startup_levels_side_by_side(emu, M, order, precision, levels):
    """A step after the first: What (two launches) and the passes of the levels.
    Level l has two passes to its first B, 2^l solves and 2^l - 1 row passes
    between them, 2^(l+1) + 1 launches: those of the longest level, or of all."""
    from emu.emu_plan import EmuPlan

    prob = periodic_problem_from_seed(190 + len(M), len(M), M, 0.01, order + 3, order=order, precision=precision)
    plan = EmuPlan(emu, prob)
    assert plan.query(Q_LEVELS) == levels
    if len(M) == 1:
        return
    plan.set_state(prob.u0)
    plan.step(1)
    L = order // 2
    passes = 2 ** L + 1 if levels > 1 else 2 ** (L + 1) - 2 + L
    assert _launches(emu, lambda: plan.step(1)) == 2 + passes


def test_batched_instances_march_their_levels_in_turn(emu):
    from emu.emu_plan import EmuBatchPlan

    prob = periodic_problem_from_seed(195, 2, (64, 64), 0.01, 10, order=8)
    assert EmuBatchPlan(emu, [prob]).query(Q_LEVELS) == 1.0
