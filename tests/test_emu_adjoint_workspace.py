"""Adjoint workspace: the complex grids it holds, counted from what a reverse
sweep keeps (u of every start-up step, the segment's B and history window, the checkpoints
of all segments but the newest, eight beta, omega of the Adams start, G of the
sub-steps, seven working grids)."""
import ctypes as C
import math

import numpy as np
import pytest

from workloads import periodic_problem_from_seed


@pytest.mark.parametrize("order, N, K", [(8, 26, 19), (8, 26, 10), (8, 26, 4), (4, 12, 100), (2, 9, 0)])
def test_workspace_holds_what_the_sweep_keeps(emu, order, N, K):
    from emu.emu_plan import EmuPlan, emu_adjoint

    M = (64, 96)
    prob = periodic_problem_from_seed(200 + order, 2, M, 0.01, N, order=order, A_kind="stepwise")
    prob.A_steps = np.random.default_rng(1).uniform(-1, 1, size=(N, 2))
    plan = EmuPlan(emu, prob)
    size = C.c_size_t()
    plan.call("tdse_adjoint_workspace_size", K, C.byref(size))
    ns, H, iters = order - 2, order - 1, N - 1 - (order - 2)
    k = K if K > 0 else math.ceil(math.sqrt(iters))
    segments = math.ceil(iters / k)
    grids = (ns + 1) + k + (k + H) + (segments - 1) * (1 + H) + 8 + H + 2 ** (order // 2 - 1) + 7
    sub_steps = 2 ** (order // 2) - 1
    tables = (16 + max(min(N - ns, 32) * 2 * H, sub_steps)) * sum(M) * 16          # phase factors
    sums = ((N - ns) * 16 + 2 * ns * sub_steps) * (M[0] * M[1] // 256 + 1) * 8     # partial sums and their totals
    rest = size.value - grids * 16 * M[0] * M[1] - tables - sums                   # lists per step, the field map
    assert 0 <= rest < 16 * M[0] * M[1]
    g, _ = emu_adjoint(plan, prob.u0, np.asarray(prob.u0) * 1j, K)
    ref, _ = emu_adjoint(plan, prob.u0, np.asarray(prob.u0) * 1j, 3)
    assert np.abs(g - ref).max() <= 1e-12 * np.abs(ref).max()
