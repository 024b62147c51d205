"""GPU parity of the adjoint's fused passes over line lengths (one wave and
several lines per workgroup, 3 * 2^a, the longest line, ragged tiles), two
potential fields, a field along both axes, and checkpoint intervals that
divide the Adams steps evenly, unevenly or not at all."""
import os

import numpy as np
import pytest

from oracle.adjoint import adjoint, dipole_seed
from oracle.periodic import PeriodicOracle
from workloads import periodic_problem_from_seed

pytestmark = pytest.mark.gpu

CASES = [((24,), 12, 8, 0), ((2048,), 12, 8, 0), ((3072,), 10, 8, 3), ((8, 1024), 10, 8, 0), ((1024, 8), 10, 6, 2),
         ((96, 48), 11, 8, 1), ((12 * 2, 768), 9, 4, 4), ((256, 256), 12, 8, 5), ((512, 1024), 8, 4, 0), ((64,), 2, 4, 0),
         ((32, 16), 3, 4, 0)]


@pytest.mark.parametrize("M, N, order, K", CASES, ids=["x".join(map(str, c[0])) + f"-{c[1]}-o{c[2]}-K{c[3]}" for c in CASES])
def test_adjoint_line_lengths(M, N, order, K):
    import torch

    from paper_2001_06113_amd import _lib
    from paper_2001_06113_amd.tdse import Plan

    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2001_06113_amd import build

        build.build()
    print(f"case adjoint M={M} steps={N} order={order} K={K}", flush=True)
    prob = periodic_problem_from_seed(170 + N, len(M), M, 0.05, N, order=order, A_kind="stepwise")
    prob.V_fields = [prob.V_fields[0], 0.3 * np.roll(prob.V_fields[0], M[0] // 3, axis=0)]
    prob.f_kind, prob.f_params = ["sin", "const"], [prob.f_params[0], (0.0, 0.0)]
    prob.A_steps = np.random.default_rng(N).uniform(-1.0, 1.0, size=(N, len(M)))
    lam = dipole_seed(prob, PeriodicOracle(prob).run()[0], axis=len(M) - 1)
    gA, g0 = adjoint(prob, lam)
    plan = Plan.from_problem(prob, device="cuda:0")
    a, b = plan.adjoint(prob.u0, lam, K)
    b = b.cpu().numpy()
    plan.close()
    assert np.max(np.abs(a - gA)) <= 1e-10 * np.max(np.abs(gA))
    assert np.linalg.norm(b - g0) <= 1e-10 * np.linalg.norm(g0)
