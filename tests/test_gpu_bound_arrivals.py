"""The FP64 bound of the quasi-Newton search where several workgroups add its terms
and the last to arrive decides: every call of many gives the first one's bounds,
steps and multipliers, bit for bit (a sum read too early, or by the wrong
workgroup, would show in one of them), and the bounds are those of the oracle."""
import numpy as np
import pytest
import torch

from gpu_common import dm, np_, say
from oracle import oracle as O
from test_gpu_bound_order import chain

pytestmark = pytest.mark.gpu


# 32, 33 and 160 blocks of 256 rows, and many blocks of exactly-one rows
@pytest.mark.parametrize("n_rows,b1_rows,long_len", [(4096, 0, 90), (4224, 0, 90), (20000, 500, 40), (3000, 0, 1)])
def test_many_calls_agree(n_rows, b1_rows, long_len):
    n, ptr, cols, coefs, rhs, cost = chain(n_rows, b1_rows, long_len, 8)
    ctx = dm().Context(0)
    ctx.build_ilp(n, ptr, cols, coefs, rhs)
    ctx.set_costs(torch.from_numpy(cost))
    say(f"  {ctx.info['n_short_rows']} + {ctx.info['n_rows'] - ctx.info['n_short_rows']} rows")
    start = ctx.dual_solve(ctx.init_lambda("fp64"), 2)[0]
    first = ctx.lbfgs_solve(start.clone(), 4)
    for _ in range(40):
        again = ctx.lbfgs_solve(start.clone(), 4)
        assert all(torch.equal(a, b) for a, b in zip(again, first))
    S = O.Space.from_ilp(n, ptr, cols, coefs, rhs)
    S.set_costs(cost)
    for lam, bound in ((start, first[1][0]), (first[0], first[1][-1])):
        a = np_(lam)
        tol = 2.0 ** -53 * (8 * len(a) * np.abs(a).max() + ctx.info["n_rows"] * np.abs(a).sum())
        assert abs(float(bound) - S.lower_bound(a)) <= tol
