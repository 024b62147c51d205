"""GPU parity of the one-workgroup 1D run over its lengths (8..2048 points, also
3 * 2^a) against the oracle, and its step-in-pieces contract bit for bit."""
import os

import numpy as np
import pytest

from oracle.periodic import PeriodicOracle
from workloads import periodic_problem_from_seed

pytestmark = pytest.mark.gpu

CASES = [(8, 8, "pulse_sin2"), (24, 6, "none"), (96, 8, "pulse_sin2"), (256, 8, "pulse_sin2"), (384, 4, "stepwise"),
         (512, 8, "none"), (768, 8, "pulse_sin2"), (1024, 8, "pulse_sin2"), (1536, 2, "pulse_sin2"), (1536, 8, "none"),
         (2048, 8, "pulse_sin2"), (2048, 4, "none")]


@pytest.mark.parametrize("M, order, A_kind", CASES, ids=[f"{c[0]}-o{c[1]}-{c[2]}" for c in CASES])
def test_run1d_lengths(M, order, A_kind):
    import torch

    from paper_2001_06113_amd import _lib
    from paper_2001_06113_amd.tdse import Plan

    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2001_06113_amd import build

        build.build()
    print(f"case run1d M={M} order={order} A={A_kind}", flush=True)
    prob = periodic_problem_from_seed(300 + M + order, 1, (M,), 0.05, order + 15, order=order, A_kind=A_kind)
    prob.V_fields = [prob.V_fields[0], 0.3 * np.roll(prob.V_fields[0], M // 3)]
    prob.f_kind, prob.f_params = ["sin", "const"], [prob.f_params[0], (0.0, 0.0)]
    plan = Plan.from_problem(prob, device="cuda:0")
    plan.profile(True)
    full = plan.run(prob.u0).cpu().numpy()
    assert plan.query(25) == 1.0 and plan.query(11) == 0.0   # one launch, no row pass
    plan.profile(False)
    plan.set_state(torch.from_numpy(np.asarray(prob.u0, dtype=np.complex128)).to("cuda:0"))
    for k in (order - 1, 1, 3, 12):
        plan.step(k)
    out = plan.get_state().cpu().numpy()
    plan.close()
    ref = PeriodicOracle(prob).run()[0]
    assert np.linalg.norm(full - ref) <= 1e-11 * np.linalg.norm(ref)
    assert np.array_equal(out, full)
