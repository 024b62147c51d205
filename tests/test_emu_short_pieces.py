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


def test_free_1d_pieces_equal_the_whole_run(emu):
    from emu.emu_plan import EmuPlan

    from workloads import free_problem_from_seed

    for M, nu, order, cheb in (((32,), (256,), 8, 0), ((40,), (512,), 4, 20), ((24,), (256,), 2, 0)):
        prob = free_problem_from_seed(60 + M[0], 1, M, 0.02, order + 14, order=order, nu=nu, eps=1e-8, q=8)
        prob.cheb = cheb
        plan = EmuPlan(emu, prob)
        full = plan.run(prob.u0)
        plan.set_state(prob.u0)
        plan.step(order)
        for k in (1, 1, 5, 1, 5):
            plan.step(k)
        plan.step(1)
        assert np.array_equal(_state(plan, M), full), (M, order)


@pytest.mark.parametrize("domain, M, order", [("periodic", 32, 8), ("periodic", 2048, 4), ("free", 32, 6)])
def test_field_changed_between_pieces(emu, domain, M, order):
    """The entries in flight are carried with the new field, as by the general
    passes (a sampled potential takes those; in free space a profiled run)."""
    from emu.emu_plan import EmuPlan

    from workloads import free_problem_from_seed

    N = order + 9
    if domain == "periodic":
        prob = periodic_problem_from_seed(150, 1, (M,), 0.05, N, order=order, A_kind="stepwise")
        prob.n_start, prob.f_kind, prob.f_params = order - 1, ["const"], [(0.0, 0.0)]
    else:
        prob = free_problem_from_seed(151, 1, (M,), 0.02, N, order=order, nu=(256,), eps=1e-8, q=8)
    rng = np.random.default_rng(7)
    fields = [np.ascontiguousarray(rng.uniform(-1, 1, size=(N, 1))) for _ in range(2)]

    prob.A_kind, prob.A_steps = "stepwise", fields[0]

    def march(plan):
        plan.call("tdse_set_field", fields[0].ctypes.data_as(C.POINTER(C.c_double)))
        plan.set_state(prob.u0)
        plan.step(order + 2)
        plan.step(1)
        plan.call("tdse_set_field", fields[1].ctypes.data_as(C.POINTER(C.c_double)))
        plan.step(1)
        plan.step(3)
        return _state(plan, prob.M)

    plan = EmuPlan(emu, prob)
    got = march(plan)
    if domain == "periodic":
        prob.V_samples, prob.V_kind = np.stack([prob.V_fields[0]] * (N + 1)), "sampled"
        ref = march(EmuPlan(emu, prob))
    else:
        plan.call("tdse_profile", 1)
        ref = march(plan)
    assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("nu, piece, six_steps", [(2048, 1, 12), (2048, 7, 12), (2048, 8, 2), (1024, 1, 2)])
def test_free_1d_path_by_the_first_piece(emu, nu, piece, six_steps):
    """Launches of a piece of six steps: two passes per step where the
    one-workgroup launch does not pay, else a phase table and one launch."""
    from emu.emu_plan import EmuPlan

    from workloads import free_problem_from_seed

    launches = C.c_int.in_dll(emu, "emu_launches")
    prob = free_problem_from_seed(63, 1, (20,), 0.02, 20, order=2, nu=(nu,), eps=1e-8, q=8)
    plan = EmuPlan(emu, prob)
    full = plan.run(prob.u0)
    plan.set_state(prob.u0)
    plan.step(piece)
    before = launches.value
    plan.step(6)
    assert launches.value - before == six_steps
    plan.step(14 - piece)
    assert np.linalg.norm(_state(plan, prob.M) - full) <= 1e-13 * np.linalg.norm(full)


@pytest.mark.parametrize("shapes, lanes", [([(64,), (64, 64)], 2), ([(64,), (64, 64), (192, 192), (64, 192)], 4)])
def test_batch_pieces_fork_their_lanes_at_most_once(emu, shapes, lanes):
    """A fork and a join are a wait per side stream each; fewer than four lanes
    stay on one stream for a single step."""
    from emu.emu_plan import EmuBatchPlan

    waits = C.c_int.in_dll(emu, "emu_event_waits")
    probs = [periodic_problem_from_seed(160 + i, len(M), M, 0.01, 6, order=2) for i, M in enumerate(shapes)]
    plan = EmuBatchPlan(emu, probs)
    full = plan.run([p.u0 for p in probs])
    packed = np.concatenate([np.asarray(p.u0, dtype=np.complex128).ravel() for p in probs])
    plan.call("tdse_set_state", C.c_void_p(packed.ctypes.data), 1)
    for k, forks in ((1, lanes == 4), (2, 2 if lanes == 4 else 0), (3, 1)):
        before = waits.value
        plan.call("tdse_step", k)
        assert waits.value - before == 2 * (lanes - 1) * forks, k
    out = np.zeros_like(packed)
    plan.call("tdse_get_state", C.c_void_p(out.ctypes.data), 1)
    assert np.array_equal(out, np.concatenate([u.ravel() for u in full]))
