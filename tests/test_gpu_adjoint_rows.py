"""GPU parity of the adjoint's fused row passes at the lengths with a schedule of their
own, 1536 and 3072 points (whole and with few lines), against the oracle."""
import os

import numpy as np
import pytest

from oracle.adjoint import adjoint, dipole_seed
from oracle.periodic import PeriodicOracle
from workloads import periodic_problem_from_seed

pytestmark = pytest.mark.gpu

CASES = [((1536,), 12, 8, 0), ((3072,), 8, 4, 2), ((8, 1536), 10, 8, 3), ((24, 3072), 9, 6, 0)]


@pytest.mark.parametrize("M, N, order, K", CASES, ids=["x".join(map(str, c[0])) for c in CASES])
def test_adjoint_long_rows(M, N, order, K):
    import torch

    from paper_2001_06113_amd import _lib
    from paper_2001_06113_amd.tdse import Plan

    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2001_06113_amd import build

        build.build()
    print(f"case adjoint rows M={M} steps={N} order={order} K={K}", flush=True)
    prob = periodic_problem_from_seed(210 + N, len(M), M, 0.02, N, order=order, A_kind="stepwise")
    prob.A_steps = np.random.default_rng(N).uniform(-1.0, 1.0, size=(N, len(M)))
    lam = dipole_seed(prob, PeriodicOracle(prob).run()[0], axis=len(M) - 1)
    gA, g0 = adjoint(prob, lam)
    plan = Plan.from_problem(prob, device="cuda:0")
    a, b = plan.adjoint(prob.u0, lam, K)
    b = b.cpu().numpy()
    plan.close()
    assert np.max(np.abs(a - gA)) <= 1e-10 * np.max(np.abs(gA))
    assert np.linalg.norm(b - g0) <= 1e-10 * np.linalg.norm(g0)
