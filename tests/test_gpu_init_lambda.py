"""First multipliers in both of their forms (an entry at a time, or a variable
at a time and then the entries): the quotient of the cost and the row count in the
message type, so the same bits as IEEE division gives, on either side of a
million entries."""
import numpy as np
import pytest
import torch

from gpu_common import dm, np_, say

pytestmark = pytest.mark.gpu


def assignment(n):
    """n x n assignment: 2 n^2 entries."""
    cells = np.arange(n * n).reshape(n, n)
    cols = np.concatenate([cells, cells.T]).ravel().astype(np.int32)
    ptr = np.arange(0, len(cols) + 1, n).astype(np.int32)
    return ptr, cols, np.ones(len(cols), np.int8), np.ones(2 * n, np.int32)


@pytest.mark.parametrize("n", [2, 90, 707, 708])   # 708^2 * 2 is the first above a million
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_quotients_are_exact(n, prec):
    ptr, cols, coefs, rhs = assignment(n)
    cost = np.random.default_rng(n).uniform(-1.0, 3.0, n * n)
    ctx = dm().Context(0)
    ctx.build_ilp(n * n, ptr, cols, coefs, rhs)
    ctx.set_costs(torch.from_numpy(cost))
    say(f"  {prec}: {ctx.info['nnz']} nonzeros")
    t = np.float32 if prec == "fp32" else np.float64
    want = (cost.astype(t) / t(2))[np_(ctx.get_space("rent_var"))]
    assert np.array_equal(np_(ctx.init_lambda(prec)), want)
