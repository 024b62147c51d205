"""Host tables of the one-launch paths: the extended-precision evaluations that
planning them takes, and the static phase factors against the exact phases of a
run without a potential."""
import ctypes as C

import numpy as np
import pytest

from workloads import periodic_problem_from_seed


def _evaluations(emu, call):
    n = C.c_int.in_dll(emu, "emu_trig")
    before = n.value
    call()
    return n.value - before


@pytest.mark.parametrize("M", [(96,), (768,), (2048,), (48, 48), (384, 384), (64, 192)])
def test_table_evaluations(emu, M):
    """A sine and a cosine per entry of each different twiddle table, one pair per
    non-negative k for the static phases; none of those for a batch's
    instances, and none at all for a new field."""
    from emu.emu_plan import EmuBatchPlan, EmuPlan

    prob = periodic_problem_from_seed(170, len(M), M, 0.02, 20, order=8, A_kind="stepwise")
    prob.A_steps = np.zeros((20, len(M)))
    plans = []
    twiddles = sum(2 * n for n in set(M if len(M) == 2 else (1,) + M))
    n = _evaluations(emu, lambda: plans.append(EmuPlan(emu, prob)))
    one_launch = plans[0].query(28) > 0
    assert one_launch == (len(M) == 1 or M[0] == M[1])
    assert n == twiddles + (M[-1] // 2 + 1 if one_launch else 0)
    assert _evaluations(emu, lambda: plans[0].call("tdse_set_field", prob.A_steps.ctypes.data_as(C.POINTER(C.c_double)))) == 0
    if min(M) >= 64 and all(m % 3 or m >= 192 for m in M):
        assert _evaluations(emu, lambda: EmuBatchPlan(emu, [prob])) == twiddles


@pytest.mark.parametrize("M, order", [((2048,), 8), ((768,), 4), ((48, 48), 8), ((64, 64), 6)])
def test_free_propagation(emu, M, order):
    """V = 0, A = 0: u(T) = F^-1 exp(-i k^2 T) F u0.  A step is two line
    transforms per axis and one product with a factor; 30 of them at 1e-15 each."""
    from emu.emu_plan import EmuPlan

    prob = periodic_problem_from_seed(171, len(M), M, 0.003, order + 8, order=order, A_kind="none")
    prob.V_fields = [np.zeros(M)]
    rng = np.random.default_rng(3)
    prob.u0 = rng.standard_normal(M) + 1j * rng.standard_normal(M)
    plan = EmuPlan(emu, prob)
    assert plan.query(28) > 0
    u = plan.run(prob.u0)
    k2 = np.zeros(M, dtype=np.longdouble)
    for a, n in enumerate(M):
        k = np.fft.fftfreq(n, 1.0 / n).astype(np.longdouble).reshape([-1 if b == a else 1 for b in range(len(M))])
        k2 = k2 + k * k
    dt = np.longdouble(prob.T / prob.nsteps)
    th = np.fmod(k2 * dt * prob.nsteps, 2 * np.arccos(np.longdouble(-1)))
    ref = np.fft.ifftn(np.fft.fftn(prob.u0) * np.exp(-1j * th).astype(np.complex128))
    assert np.linalg.norm(u - ref) <= 3e-14 * np.linalg.norm(ref)
