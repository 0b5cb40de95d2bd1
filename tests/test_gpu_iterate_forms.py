"""The forms of the hard iteration by problem size, on 0-1 ILPs that mix every
kind of row (tiles of each width, chunks with and without a right-hand side, and
exactly-one rows from 4 to 1500 entries), step by step against the FP64 oracle.

u = 2^-24 or 2^-53.  One iteration takes an entry through fewer than 100
roundings of values at most a few times the largest multiplier: its result is
within 300 u of that.  A bound of given multipliers: each restored one is within
8 u of its size, and a row adds at most 2 more roundings for each of its own, so
the bound is within 10 u of their absolute sum: far below any row's own term."""
import numpy as np
import pytest
import torch

from gpu_common import dm, np_, say
from oracle import oracle as O

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 0), (3, 3, 0), (3, 4, 0), (5, 5, 0), (6, 5, 0), (8, 8, 0), (9, 8, 0), (4, 4, 1), (2, 5, -1), (14, 13, 0)]


def mixed(lens, n_side, seed):
    """Exactly-one rows of the given lengths and n_side rows of SHAPES in turn
    over shared variables, each in at most three of the former and two of the
    latter; every exactly-one row and every unit of a right-hand side has a
    private variable, and those alone satisfy the rows."""
    rng = np.random.default_rng([len(lens), sum(lens), n_side, seed])
    short = [SHAPES[i % len(SHAPES)] for i in range(n_side)]
    m = max(max(lens, default=0), sum(lens) // 3, sum(p + q for p, q, _ in short) // 2, 30) + 30
    rows, n = [], m

    def pools(k):   # every variable at most k times, no row twice the same one
        order, at = np.concatenate([rng.permutation(m) for _ in range(k)]), 0
        while True:
            size = yield
            v = np.unique(order[at:at + size])
            at += size
            yield v

    take = pools(3)
    for length in lens:
        next(take)
        v = take.send(length - 1)
        rows.append((np.append(v, n), np.ones(len(v) + 1, int), 1))
        n += 1
    take = pools(2)
    for p, q, b in short:
        next(take)
        v = take.send(p + q - abs(b))
        c = np.resize([1, -1], len(v))
        c[:p - max(b, 0)], c[p - max(b, 0):] = 1, -1
        v, c = np.append(v, np.arange(n, n + abs(b))), np.append(c, np.full(abs(b), np.sign(b)))
        n += abs(b)
        o = rng.permutation(len(v))
        rows.append((v[o], c[o], b))
    used = np.unique(np.concatenate([r[0] for r in rows]))
    new = np.full(n, -1)
    new[used] = np.arange(len(used))
    ptr = np.cumsum([0] + [len(r[0]) for r in rows]).astype(np.int32)
    cols = new[np.concatenate([r[0] for r in rows])].astype(np.int32)
    coefs = np.concatenate([r[1] for r in rows]).astype(np.int8)
    return len(used), ptr, cols, coefs, np.array([r[2] for r in rows], np.int32), rng.uniform(-0.5, 1.0, len(used))


MIDDLE = [([40] * 145, 60),              # just over what one workgroup takes
          ([4, 90, 300] * 40, 200),      # a wave per exactly-one row
          ([520, 1500] * 12, 120),       # a block per exactly-one row, entries beyond the registers
          ([], 1500),                    # none of them
          ([250] * 640, 900)]            # 170k entries, the largest such problems
# one workgroup: 4, 16 and 64 lanes per exactly-one row, entries beyond a lane's registers
SMALL = [([10] * 40, 60), ([30] * 30, 40), ([5, 7, 160] * 8, 10), ([300] * 8, 0), ([300, 70] * 6, 40), ([100, 400] * 4, 60),
         ([], 300)]
LARGE = [([260] * 700, 900)]             # two passes


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("lens,n_side", MIDDLE + SMALL + LARGE)
def test_steps_match_the_oracle(lens, n_side, prec):
    n, ptr, cols, coefs, rhs, cost = mixed(lens, n_side, 1)
    S = O.Space.from_ilp(n, ptr, cols, coefs, rhs)
    S.set_costs(cost)
    ctx = dm().Context(0)
    ctx.build_ilp(n, ptr, cols, coefs, rhs)
    ctx.set_costs(torch.from_numpy(cost))
    say(f"  {prec}: {ctx.info['n_short_rows']} + {ctx.info['n_rows'] - ctx.info['n_short_rows']} rows, "
        f"{ctx.info['nnz']} nonzeros of {ctx.info['n_free']} variables")
    assert ctx.info["nnz"] == S.info["nnz"] > 0
    u = 2.0 ** -24 if prec == "fp32" else 2.0 ** -53
    at = [ctx.init_lambda(prec)]
    for k in range(4):
        lam, trace = ctx.dual_solve(at[k].clone(), 1)
        a, b = np_(at[k]).astype(np.float64), np_(lam).astype(np.float64)
        want, _ = S.dual_solve(1, lam=a)
        assert np.abs(b - want).max() <= 300 * u * np.abs(a).max()
        assert abs(float(trace[0]) - S.lower_bound(a)) <= 10 * u * np.abs(a).sum()
        at.append(lam)
    for iters in (3, 4):   # an odd and an even number in one call
        lam, trace = ctx.dual_solve(at[0].clone(), iters)
        end, top = np_(at[iters]).astype(np.float64), np.abs(np_(at[iters])).max()
        # the steps above restore feasibility once more each (8 u); a step at most triples a difference
        assert np.abs(np_(lam).astype(np.float64) - end).max() <= 8 * 3 ** iters * u * top
        for k in range(iters):
            a = np_(at[k]).astype(np.float64)
            assert abs(float(trace[k]) - S.lower_bound(a)) <= (10 + 8 * 3 ** k) * u * np.abs(a).sum()
        again = ctx.dual_solve(at[0].clone(), iters, trace=False)[0]
        assert torch.equal(again, lam)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_both_buffers_in_a_workspace(prec):
    """One launch per iteration alternates between two cell buffers, the context's
    own or those of a workspace, here full of NaN, of which nothing is used once it
    is detached."""
    n, ptr, cols, coefs, rhs, cost = mixed([40] * 145, 60, 2)
    ctx = dm().Context(0)
    ctx.build_ilp(n, ptr, cols, coefs, rhs)
    ctx.set_costs(torch.from_numpy(cost))
    start = ctx.init_lambda(prec)
    none = ctx.dual_solve(start.clone(), 0)[0]
    bound = ctx.lower_bound(start)
    own = {k: ctx.dual_solve(start.clone(), k) for k in (1, 2, 5)}
    assert float(own[1][1][0]) == pytest.approx(bound, rel=1e-12)
    ws = torch.full((ctx.workspace_bytes(prec),), 255, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(prec, ws)
    for k in (5, 1, 2):
        lam, trace = ctx.dual_solve(start.clone(), k)
        assert torch.equal(lam, own[k][0]) and torch.equal(trace, own[k][1])
    ctx.set_workspace(prec, None)
    torch.cuda.synchronize()
    kept = ws.fill_(255).clone()
    assert torch.equal(ctx.dual_solve(start.clone(), 0)[0], none)
    for k in (2, 5, 1):
        lam, trace = ctx.dual_solve(start.clone(), k)
        assert torch.equal(lam, own[k][0]) and torch.equal(trace, own[k][1])
    torch.cuda.synchronize()
    assert torch.equal(ws, kept)
