"""CPU run of the adjoint's fused row passes at the lengths with a schedule of their
own, 1536 and 3072 points (whole and with few lines), against the oracle."""
import numpy as np
import pytest

from oracle.adjoint import adjoint, dipole_seed
from oracle.periodic import PeriodicOracle
from workloads import periodic_problem_from_seed

CASES = [((1536,), 6, 4, 2), ((8, 3072), 4, 2, 0)]


@pytest.mark.parametrize("M, N, order, K", CASES, ids=["x".join(map(str, c[0])) for c in CASES])
def test_adjoint_long_rows(emu, M, N, order, K):
    from emu.emu_plan import EmuPlan, emu_adjoint

    prob = periodic_problem_from_seed(210 + N, len(M), M, 0.02, N, order=order, A_kind="stepwise")
    prob.A_steps = np.random.default_rng(N).uniform(-1.0, 1.0, size=(N, len(M)))
    lam = dipole_seed(prob, PeriodicOracle(prob).run()[0], axis=len(M) - 1)
    gA, g0 = adjoint(prob, lam)
    a, b = emu_adjoint(EmuPlan(emu, prob), prob.u0, lam, K)
    assert np.max(np.abs(a - gA)) <= 1e-10 * np.max(np.abs(gA))
    assert np.linalg.norm(b - g0) <= 1e-10 * np.linalg.norm(g0)
