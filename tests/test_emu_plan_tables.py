"""Host tables of the one-launch paths: what planning them costs beside a plan
that does not have them (the split form of the same grid), and the static phase
factors against the exact phases of a run without a potential."""
import ctypes as C
import time

import numpy as np
import pytest

from workloads import periodic_problem_from_seed


def _plan_ms(lib, prob):
    from paper_2001_06113_amd.tdse import problem_kwargs, problem_struct

    struct, keep = problem_struct(**problem_kwargs(prob))
    best = float("inf")
    for _ in range(40):
        h = C.c_void_p()
        t0 = time.perf_counter()
        assert lib.tdse_plan(C.byref(struct), C.byref(h)) == 0
        best = min(best, time.perf_counter() - t0)
        lib.tdse_destroy(h)
    return 1e3 * best


@pytest.mark.parametrize("M, factor", [((768,), 1.6), ((2048,), 1.6), ((384, 384), 2.0)])
def test_planning_time(emu, M, factor):
    probs = [periodic_problem_from_seed(170, len(M), M, 0.02, 100, precision=p) for p in ("fp64", "fp32split")]
    one, plain = (_plan_ms(emu, p) for p in probs)
    print(f"plan {M}: {one:.3f} ms, without the tables {plain:.3f} ms")
    assert one <= factor * plain


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
