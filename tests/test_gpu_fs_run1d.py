"""GPU: the one-workgroup 1D free-space run over its points per thread (M up to
nu), orders, the interpolant and the longest line: the path is the one taken,
agrees with the oracle and the general passes, and its pieces are the whole run
bit for bit."""
import os

import numpy as np
import pytest

from oracle.freespace import FreeSpaceOracle
from workloads import free_problem_from_seed

pytestmark = pytest.mark.gpu

CASES = [(30, 256, 8, 0), (60, 256, 6, 0), (100, 256, 4, 0), (140, 256, 8, 0), (100, 1024, 8, 0), (40, 512, 2, 20),
         (256, 2048, 8, 0)]


@pytest.mark.parametrize("M, nu, order, cheb", CASES, ids=[f"{c[0]}-nu{c[1]}-o{c[2]}-c{c[3]}" for c in CASES])
def test_free_1d_run(M, nu, order, cheb):
    import torch

    from paper_2001_06113_amd import _lib
    from paper_2001_06113_amd.tdse import Q_PATH, Plan

    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2001_06113_amd import build

        build.build()
    print(f"case 1D free-space run M={M} nu={nu} order={order} cheb={cheb}", flush=True)
    prob = free_problem_from_seed(180 + M, 1, (M,), 0.01, order + 20, order=order, nu=(nu,), eps=1e-8, q=8)
    prob.cheb = cheb
    plan = Plan.from_problem(prob, device="cuda:0")
    assert plan.query(Q_PATH) == 3.0
    u = plan.run(prob.u0).cpu().numpy()
    plan.set_state(prob.u0)
    for k in (order + 4, 1, 1, 6, 8):
        plan.step(k)
    pieces = plan.get_state().cpu().numpy()
    assert plan.query(Q_PATH) == 3.0
    plan.profile(True)
    plan.set_state(prob.u0)
    assert plan.query(Q_PATH) == 0.0
    two = plan.run(prob.u0).cpu().numpy()
    plan.close()
    assert np.linalg.norm(u - FreeSpaceOracle(prob).run()[0]) <= 1e-11 * np.linalg.norm(u)
    assert np.linalg.norm(u - two) <= 1e-12 * np.linalg.norm(u)
    assert np.array_equal(pieces, u)
