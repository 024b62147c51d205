"""GPU parity of the FP64 passes over lengths 3 * 2^a (24..768 points: rows,
columns and the middle axis) against the oracle: ragged sets of lines, two
potential fields, a field along every axis, low orders.  (The adjoint has row
passes of its own; its recomputation takes these.)"""
import os

import numpy as np
import pytest

from oracle.periodic import PeriodicOracle
from workloads import periodic_problem_from_seed

pytestmark = pytest.mark.gpu

CASES = [((24,), 12, 8), ((192,), 10, 6), ((768,), 12, 8), ((768, 8), 9, 4), ((8, 768), 10, 8), ((48, 96), 12, 8),
         ((384, 24), 10, 8), ((192, 384), 9, 8), ((16, 48, 24), 9, 8), ((24, 96, 8), 6, 4), ((8, 24, 192), 5, 2)]


@pytest.mark.parametrize("M, N, order", CASES, ids=["x".join(map(str, c[0])) + f"-o{c[2]}" for c in CASES])
def test_three_smooth_lengths(M, N, order):
    import torch

    from paper_2001_06113_amd import _lib
    from paper_2001_06113_amd.tdse import CFG_PERSISTENT, Plan

    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2001_06113_amd import build

        build.build()
    print(f"case three-smooth M={M} steps={N} order={order}", flush=True)
    prob = periodic_problem_from_seed(210 + M[0], len(M), M, 1e-3 * N, N, order=order)
    prob.A_params = prob.A_params[:3] + (0.6, -0.8, 0.5)[:len(M)]
    prob.V_fields = [prob.V_fields[0], 0.3 * np.roll(prob.V_fields[0], M[0] // 3, axis=0)]
    prob.f_kind, prob.f_params = ["sin", "const"], [prob.f_params[0], (0.0, 0.0)]
    plan = Plan.from_problem(prob, device="cuda:0")
    plan.configure(CFG_PERSISTENT, 0)
    u = plan.run(prob.u0).cpu().numpy()
    plan.close()
    ref = PeriodicOracle(prob).run()[0]
    assert np.linalg.norm(u - ref) <= 1e-11 * np.linalg.norm(ref)
