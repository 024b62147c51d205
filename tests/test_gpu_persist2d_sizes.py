"""GPU parity of the persistent 2D Adams steps at lengths 3 * 2^a, and of many
short launches in a row (each launch marks its exchange buffers anew)."""
import os

import numpy as np
import pytest

from oracle.periodic import PeriodicOracle
from workloads import periodic_problem_from_seed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2001_06113_amd import _lib

    if not os.path.exists(_lib.LIB_PATH):
        from paper_2001_06113_amd import build

        build.build()
    yield


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def _plan(M, steps, order, dir2):
    from paper_2001_06113_amd.tdse import Q_PATH, Plan

    prob = periodic_problem_from_seed(47 + M, 2, (M, M), 1e-3 * steps, steps, order=order)
    if dir2:
        prob.A_params = prob.A_params[:3] + (0.6, -0.8)
    plan = Plan.from_problem(prob, device="cuda:0")
    assert plan.query(Q_PATH) == 2.0
    return prob, plan


@pytest.mark.parametrize("M, steps, order, dir2", [(48, 20, 8, True), (96, 30, 4, False), (192, 25, 6, True),
                                                   (384, 20, 8, True), (384, 20, 8, False)])
def test_persistent_three_smooth_sizes(M, steps, order, dir2):
    print(f"case persistent 2D M={M} steps={steps} order={order} dir2={dir2}", flush=True)
    prob, plan = _plan(M, steps, order, dir2)
    r = rel(plan.run(prob.u0).cpu().numpy(), PeriodicOracle(prob).run()[0])
    plan.close()
    assert r <= 1e-11


@pytest.mark.parametrize("M", [32, 96])
def test_persistent_single_steps_equal_one_run(M):
    print(f"case persistent 2D one step at a time M={M}", flush=True)
    prob, plan = _plan(M, 40, 8, True)
    full = plan.run(prob.u0).cpu().numpy()
    plan.set_state(prob.u0)
    for _ in range(40):
        plan.step(1)
    got = plan.get_state().cpu().numpy()
    plan.close()
    assert np.array_equal(got, full)


def test_steps_under_capture_take_the_passes():
    import torch

    print("case 96^2 steps captured by the caller", flush=True)
    prob, plan = _plan(96, 16, 8, True)
    ref = plan.run(prob.u0).clone()
    u0 = torch.as_tensor(prob.u0).to("cuda:0")
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(g, stream=side):
        plan.set_state(u0)
        plan.step(16)
        out = plan.get_state()
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert (torch.linalg.vector_norm(out - ref) / torch.linalg.vector_norm(ref)).item() <= 1e-13
    plan.close()
