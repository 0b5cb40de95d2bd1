"""Smoothed rows at temperatures so small against the multipliers that their
quotient comes near the type's largest number (FP32: values of 1e33 to 1e38
temperatures): every finite partial sum counts, as in FP64.

With u = 2^-24 or 2^-53, an iteration takes an entry through fewer than 100
roundings of values at most a few times the largest cost (the soft-mins' own
terms, at most T log 25, vanish beside them), so three leave at most 1e-4 or
1e-12 of it.  The bound of given multipliers: each restored one is within 8 u of
the largest, and the entry sums of a row pass 2 more roundings each."""
import numpy as np
import pytest
import torch

from gpu_common import both, dm, np_, say
from oracle import oracle as O
from synth import make_pair
from test_gpu_row_forms import rows_of_one_shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,T", [("fp32", 4e-37), ("fp32", 1e-34), ("fp32", 1e-30), ("fp64", 4e-307),
                                    ("fp64", 1e-304)])
@pytest.mark.parametrize("p,q,n_rows,b", [(3, 3, 64, 0), (4, 3, 33, 1), (7, 8, 40, 0), (12, 12, 9, 0), (10, 9, 12, -2)])
def test_tiny_temperatures_match_the_oracle(p, q, n_rows, b, prec, T):
    n, ptr, cols, coefs, rhs, cost = rows_of_one_shape(p, q, n_rows, b, 2)
    S = O.Space.from_ilp(n, ptr, cols, coefs, rhs)
    S.set_costs(cost)
    ctx = dm().Context(0)
    ctx.build_ilp(n, ptr, cols, coefs, rhs)
    ctx.set_costs(torch.from_numpy(cost))
    say(f"  p={p} q={q} b={b} {prec} T={T}: longest row {ctx.info['max_short_row']}, {ctx.info['nnz']} nonzeros")
    scale = np.abs(cost).max()
    tol, u = (1e-4, 2.0 ** -24) if prec == "fp32" else (1e-12, 2.0 ** -53)
    lam, _ = ctx.dual_solve(ctx.init_lambda(prec), 3, temperature=T)
    rlam, _ = S.dual_solve(3, T=T)
    assert np.abs(np_(lam) - rlam).max() <= tol * scale
    at = np_(lam).astype(np.float64)
    assert abs(ctx.lower_bound(lam, T) - S.lower_bound(at, T)) <= 10 * u * len(at) * np.abs(at).max()


@pytest.mark.parametrize("T", [4e-37, 1e-34])
def test_marginals_at_a_tiny_temperature_are_the_minimisers(T):
    pair = make_pair(1, 0, desc_noise=1.0)
    _, ctx = both(pair, 16, "fp32")
    torch.manual_seed(3)
    lam = ctx.init_lambda("fp32")
    lam += 0.1 * torch.randn(len(lam), device=lam.device)   # no two assignments of a row agree
    g, _ = ctx.subgradient(lam)
    DX, DY = torch.from_numpy(pair.DX), torch.from_numpy(pair.DY)
    gc = np_(ctx.smoothed_backward(lam, T, DX, DY)[0])
    var, n = np_(ctx.get_space("rent_var")), ctx.info["n_free"]
    deg = np.bincount(var, minlength=n)
    want = np.bincount(var, weights=np_(g), minlength=n) / deg
    assert np.abs(gc[np_(ctx.get_space("free_var"))] - want).max() <= 1e-6   # at most five ones over |J|, in FP32
