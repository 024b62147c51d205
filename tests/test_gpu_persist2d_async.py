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


def test_a_run_captured_while_steps_are_under_way():
    """The captured run takes the passes and does not wait for the launch."""
    import torch

    from paper_2001_06113_amd.tdse import CFG_PERSISTENT, Plan

    print("case capture behind persistent steps 96^2", flush=True)
    prob = periodic_problem_from_seed(135, 2, (96, 96), 0.02, 16, order=8)
    plan = Plan.from_problem(prob, device="cuda:0")
    u0 = torch.as_tensor(prob.u0).to("cuda:0", torch.complex128)
    ref = plan.run(u0).clone()
    plan.set_state(u0)
    plan.step(16)
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(g, stream=side):
        out = plan.run(u0)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert (torch.linalg.vector_norm(out - ref) / torch.linalg.vector_norm(ref)).item() <= 1e-13
    plan.configure(CFG_PERSISTENT, 0)
    assert torch.equal(plan.run(u0), out)
    plan.close()


@pytest.mark.parametrize("M", [64, 384])
def test_plans_on_streams_of_their_own(M):
    """Steps of three plans, queued without waiting: their launches take turns."""
    import torch

    from paper_2001_06113_amd.tdse import Plan

    print(f"case persistent plans on three streams M={M}", flush=True)
    probs = [periodic_problem_from_seed(140 + i, 2, (M, M), 0.02, 40, order=8) for i in range(3)]
    plans = [Plan.from_problem(p, device="cuda:0") for p in probs]
    u0 = [torch.as_tensor(p.u0).to("cuda:0", torch.complex128) for p in probs]
    ref = [p.run(u).clone() for p, u in zip(plans, u0)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in plans]
    out = [None] * 3
    for k in (20, 1, 19):
        for i, plan in enumerate(plans):
            with torch.cuda.stream(streams[i]):
                if k == 20:
                    plan.set_state(u0[i])
                plan.step(k)
                if k == 19:
                    out[i] = plan.get_state()
    torch.cuda.synchronize()
    for plan, a, b in zip(plans, out, ref):
        assert torch.equal(a, b)
        plan.close()
