"""Row forms of the hard sweep: one lane per row in tiles of each width, one
lane per entry in chunks, projection rows, and variables in one to five rows.

Generic 0-1 ILPs whose other rows all have one shape (p entries +1, q entries
-1) on either side of the tile widths, in numbers that leave ragged 64-row
tiles and below and above the size that one workgroup takes, against the FP64 oracle: multipliers and bounds after six Jacobi
iterations, the bound alone, and the row minimisers.  An iteration takes an
entry through fewer than 100 roundings of values at most a few times the
largest cost, so six leave at most 600 units in the last place, 2^-53 or 2^-24
of that scale: below 1e-12 and 1e-4 of the largest cost."""
import numpy as np
import pytest
import torch

from gpu_common import dm, np_, say
from oracle import oracle as O

pytestmark = pytest.mark.gpu


def rows_of_one_shape(p, q, n_rows, b, seed):
    """n_rows rows with p entries +1 and q entries -1 and right-hand side b,
    each variable in one to three of them, and exactly-one rows of 2 to 90
    variables over most of the variables; satisfied by x = 1 on every
    exactly-one row's first variable (outside the other rows) and, for b, on b
    private variables of each row."""
    rng = np.random.default_rng([p, q, n_rows, b + 8, seed])
    m = max(p + q, (p + q) * n_rows // 2)
    rows, n = [], m
    uses = np.zeros(m, int)
    for _ in range(n_rows):
        pool = np.flatnonzero(uses < 3)
        v = rng.choice(pool, p + q - abs(b), replace=False) if len(pool) >= p + q else rng.choice(m, 0)
        if len(v) == 0 and p + q > abs(b):
            continue
        uses[v] += 1
        own = np.arange(n, n + abs(b))
        n += abs(b)
        v = np.concatenate([own, v])
        c = np.concatenate([np.full(abs(b), np.sign(b)), np.full(p - max(b, 0), 1), np.full(q - max(-b, 0), -1)])
        o = rng.permutation(len(v))
        rows.append((v[o], c[o].astype(int), b))
    order, at = rng.permutation(m), 0
    while at < m - 2:
        k = int(rng.choice([1, 2, 5, 20, 89]))
        rows.append((np.concatenate([[n], order[at:at + k]]), np.ones(len(order[at:at + k]) + 1, int), 1))
        n += 1
        at += k + int(rng.integers(2))
    used = np.unique(np.concatenate([r[0] for r in rows]))
    new = np.full(n, -1)
    new[used] = np.arange(len(used))
    ptr = np.cumsum([0] + [len(r[0]) for r in rows]).astype(np.int32)
    cols = new[np.concatenate([r[0] for r in rows])].astype(np.int32)
    coefs = np.concatenate([r[1] for r in rows]).astype(np.int8)
    return len(used), ptr, cols, coefs, np.array([r[2] for r in rows], np.int32), rng.uniform(-0.5, 1.0, len(used))


@pytest.mark.parametrize("p,q,n_rows,b", [(1, 1, 1, 0), (3, 3, 64, 0), (3, 4, 65, 0), (5, 2, 63, 0), (5, 5, 257, 0),
                                          (6, 5, 130, 0), (8, 8, 64, 0), (8, 9, 70, 0), (30, 30, 9, 0), (4, 4, 40, 1),
                                          (3, 5, 40, -2), (3, 3, 800, 0), (3, 3, 560, 0),
                                          (2, 2, 3000, 0), (8, 7, 2100, 0)])
def test_rows_of_every_form_match_the_oracle(p, q, n_rows, b):
    n, ptr, cols, coefs, rhs, cost = rows_of_one_shape(p, q, n_rows, b, 1)
    S = O.Space.from_ilp(n, ptr, cols, coefs, rhs)
    S.set_costs(cost)
    ctx = dm().Context(0)
    ctx.build_ilp(n, ptr, cols, coefs, rhs)
    ctx.set_costs(torch.from_numpy(cost))
    say(f"  p={p} q={q} b={b}: {ctx.info['n_short_rows']} + {ctx.info['n_rows'] - ctx.info['n_short_rows']} rows, "
        f"{ctx.info['nnz']} nonzeros")
    assert ctx.info["nnz"] == S.info["nnz"] > 0
    scale = np.abs(cost).max()
    for prec, tol in (("fp64", 1e-12), ("fp32", 1e-4)):
        lam, tr = ctx.dual_solve(ctx.init_lambda(prec), 6)
        rlam, rtr = S.dual_solve(6)
        assert np.abs(np_(lam) - rlam).max() <= tol * scale
        assert np.abs(np_(tr) - rtr).max() <= tol * scale * ctx.info["n_rows"]
        again = ctx.dual_solve(ctx.init_lambda(prec), 6, trace=False)[0]
        assert torch.equal(again, lam)
        ctx.timing(True)
        ctx.dual_solve(ctx.init_lambda(prec), 6)
        assert ctx.timing_read()[0] == 6   # iterations, however they were launched
        ctx.timing(False)
        assert abs(ctx.lower_bound(lam) - S.lower_bound(rlam)) <= tol * scale * ctx.info["n_rows"]
    g, _ = ctx.subgradient(ctx.init_lambda("fp64"))   # no two multipliers agree there
    assert np.array_equal(np_(g), S.subgradient(S.init_lambda()))
