"""GPU: a persistent 2D step does not wait for the stream it is bound to (lengths
2^a and 3 * 2^a), and its result is the oracle's."""
import os

import numpy as np
import pytest

from oracle.periodic import PeriodicOracle
from workloads import periodic_problem_from_seed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [64, 96])
def test_steps_are_asynchronous(M):
    import torch

    from paper_2001_06113_amd import _lib
    from paper_2001_06113_amd.tdse import Q_PATH, Plan

    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2001_06113_amd import build

        build.build()
    print(f"case asynchronous persistent steps M={M}", flush=True)
    prob = periodic_problem_from_seed(130 + M, 2, (M, M), 0.02, 20, order=8)
    plan = Plan.from_problem(prob, device="cuda:0")
    assert plan.query(Q_PATH) == 2.0
    first = plan.run(prob.u0).cpu().numpy()
    u0 = torch.as_tensor(prob.u0).to("cuda:0", torch.complex128)
    with torch.cuda.stream(plan.stream):
        torch.cuda._sleep(200_000_000)   # some tenths of a second of work ahead of the steps
    plan.set_state(u0)
    for k in (7, 1, 12):
        plan.step(k)
    out = plan.get_state()
    assert not plan.stream.query()       # still under way
    out = out.cpu().numpy()
    plan.close()
    ref = PeriodicOracle(prob).run()[0]
    assert np.linalg.norm(out - ref) <= 1e-11 * np.linalg.norm(ref)
    assert np.array_equal(out, first)
