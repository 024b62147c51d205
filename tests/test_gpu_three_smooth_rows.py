"""GPU parity of 3 * 2^a rows on either side of the lines from which the FP64
passes take one element layout instead of two: sub-steps (P = 3 * 2^18 modes from
384 points on, 3 * 2^19 below) and Adams steps with a field along the rows."""
import os

import numpy as np
import pytest

from oracle.periodic import PeriodicOracle
from workloads import periodic_problem_from_seed

pytestmark = pytest.mark.gpu

CASES = [(8, 128, 768), (8, 256, 384), (8, 384, 384), (16, 1024, 96), (64, 128, 192)]


@pytest.mark.parametrize("M", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_many_rows(M):
    import torch

    from paper_2001_06113_amd import _lib
    from paper_2001_06113_amd.tdse import Plan

    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2001_06113_amd import build

        build.build()
    print(f"case many three-smooth rows M={M}", flush=True)
    prob = periodic_problem_from_seed(220, 3, M, 4e-3, 5, order=4)
    prob.A_params = prob.A_params[:3] + (0.6, -0.8, 0.5)
    plan = Plan.from_problem(prob, device="cuda:0")
    u = plan.run(prob.u0).cpu().numpy()
    plan.close()
    ref = PeriodicOracle(prob).run()[0]
    assert np.linalg.norm(u - ref) <= 1e-11 * np.linalg.norm(ref)
