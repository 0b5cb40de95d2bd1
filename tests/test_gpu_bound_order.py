"""The FP64 bounds of the quasi-Newton search, whose terms are added in an order
of the problem's own: every row's term once, whichever way the places were found
(few rows by counting, many by sorting) and the terms added (by the search's own
workgroup or in a launch before it).

Oracle: the FP64 bound of the same multipliers.  With u = 2^-53 each restored
multiplier is within 8 u of the largest, so are the nnz summands of the row
minima, and adding n rows' terms in any order loses at most n u of their
absolute sum, which the multipliers' bounds."""
import numpy as np
import pytest
import torch

from gpu_common import dm, np_, say
from oracle import oracle as O

pytestmark = pytest.mark.gpu


def chain(n_rows, b1_rows, long_len, seed):
    """n_rows rows x_2i + x_2i+1 = x_2i+2 + x_2i+3, b1_rows rows x_j + y_j = 1 +
    z_j over private y and z, and exactly-one rows of long_len consecutive
    variables and a private one; satisfied by the private variables alone."""
    m = 2 * n_rows + 2
    i = 2 * np.arange(n_rows)[:, None]
    rows = [(np.concatenate([r, r + 2]), [1, 1, -1, -1], 0) for r in (i + np.arange(2))]
    n = m
    for j in range(b1_rows):
        rows.append((np.array([j, n, n + 1]), [1, 1, -1], 1))
        n += 2
    for a in range(0, m - 1, long_len):
        v = np.arange(a, min(a + long_len, m))
        rows.append((np.append(v, n), [1] * (len(v) + 1), 1))
        n += 1
    ptr = np.cumsum([0] + [len(r[0]) for r in rows]).astype(np.int32)
    cols = np.concatenate([r[0] for r in rows]).astype(np.int32)
    coefs = np.concatenate([r[1] for r in rows]).astype(np.int8)
    cost = np.random.default_rng(seed).uniform(-0.5, 1.0, n)
    return n, ptr, cols, coefs, np.array([r[2] for r in rows], np.int32), cost


@pytest.mark.parametrize("n_rows,b1_rows,long_len", [(1, 0, 4), (64, 3, 20), (257, 0, 100), (2000, 260, 5),
                                                     (8192, 0, 1500), (8100, 90, 90), (8193, 0, 700),
                                                     (16384, 0, 30), (16300, 90, 8), (20000, 500, 1)])
def test_every_term_is_added_once(n_rows, b1_rows, long_len):
    n, ptr, cols, coefs, rhs, cost = chain(n_rows, b1_rows, long_len, 3)
    S = O.Space.from_ilp(n, ptr, cols, coefs, rhs)
    S.set_costs(cost)
    ctx = dm().Context(0)
    ctx.build_ilp(n, ptr, cols, coefs, rhs)
    ctx.set_costs(torch.from_numpy(cost))
    lam, _ = ctx.dual_solve(ctx.init_lambda("fp64"), 3)
    ref = np_(lam).copy()
    say(f"  {ctx.info['n_short_rows']} + {ctx.info['n_rows'] - ctx.info['n_short_rows']} rows, {ctx.info['nnz']} nonzeros")
    assert ctx.info["nnz"] == len(ref) > 0
    tol = 2.0 ** -53 * (8 * len(ref) * np.abs(ref).max() + ctx.info["n_rows"] * np.abs(ref).sum())
    _, trace, _, _ = ctx.lbfgs_solve(lam, 3)
    assert abs(np_(trace)[0] - S.lower_bound(ref)) <= tol
    end = np_(lam)
    tol = 2.0 ** -53 * (8 * len(ref) * np.abs(end).max() + ctx.info["n_rows"] * np.abs(end).sum())
    assert abs(np_(trace)[-1] - S.lower_bound(end)) <= tol


@pytest.mark.parametrize("iters", [0, 1, 300])
def test_no_rows_left(iters):
    """Presolve fixes every variable: each bound is the constant, exactly."""
    ctx = dm().Context(0)
    ctx.build_ilp(2, np.array([0, 1, 3], np.int32), np.array([0, 0, 1], np.int32), np.ones(3, np.int8),
                  np.ones(2, np.int32))
    ctx.set_costs(torch.tensor([0.75, 5.0], dtype=torch.float64))
    assert ctx.info["nnz"] == 0
    for prec in ("fp64", "fp32"):
        lam, trace = ctx.dual_solve(ctx.init_lambda(prec), iters)
        assert lam.numel() == 0 and np.array_equal(np_(trace), np.full(iters, 0.75))
        assert ctx.lower_bound(lam) == 0.75
