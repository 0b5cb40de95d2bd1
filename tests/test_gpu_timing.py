"""dm_timing_*: every sweep of every entry point is timed and counted once, in
whichever kernels it runs, and their durations together fit the call."""
import time

import pytest
import torch

from gpu_common import dm, say
from test_gpu_row_forms import rows_of_one_shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(3, 3, 64), (3, 3, 2000)])   # one workgroup takes the iterations of the first
def test_every_sweep_is_counted(shape, prec):
    n, ptr, cols, coefs, rhs, cost = rows_of_one_shape(*shape, 0, 5)
    ctx = dm().Context(0)
    ctx.build_ilp(n, ptr, cols, coefs, rhs)
    ctx.set_costs(torch.from_numpy(cost))
    lam = ctx.dual_solve(ctx.init_lambda(prec), 4)[0]
    rounds = ctx.round_primal(lam, rounds=2, iters_per_round=3)[3]
    calls = {
        "dual_solve": (lambda: ctx.dual_solve(lam.clone(), 7), 7),
        "smoothed dual_solve": (lambda: ctx.dual_solve(lam.clone(), 5, temperature=0.1), 5),
        "lower_bound": (lambda: ctx.lower_bound(lam), 1),
        "smoothed lower_bound": (lambda: ctx.lower_bound(lam, 0.1), 1),
        "subgradient": (lambda: ctx.subgradient(lam), 1),
        # two probes, the update and the subgradient an iteration, and one at the start
        "lbfgs_solve": (lambda: ctx.lbfgs_solve(lam.clone(), 3, max_search=1), 1 + 3 * 4),
        "confident_fixing": (lambda: ctx.confident_fixing(lam, 0.5), 1),
        # an evaluation before every round and after the last, three iterations a round
        "round_primal": (lambda: ctx.round_primal(lam, rounds=2, iters_per_round=3), 1 + 4 * rounds),
    }
    for name, (call, sweeps) in calls.items():
        ctx.timing(True)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        call()
        count, ms = ctx.timing_read()
        wall = 1e3 * (time.perf_counter() - t0)
        ctx.timing(False)
        say(f"  {shape} {prec} {name}: {count} sweeps, {ms:.4f} ms of {wall:.3f}")
        assert count == sweeps, name
        assert 0.0 < ms < wall, name
    call()
    assert ctx.timing_read() == (0, 0.0)
