"""Candidate lists at the sizes where their kernels change form: rows that
just fill a block's registers (2048 values) and one more, ragged 64-row
tiles, descriptor widths around the LDS stages (32, 128), K from 1 to the
whole row, and ties, against a stable sort of the FP32 squared distances
summed in the same order.  The distances are formed by the same fused
multiply-adds, so the lists are equal exactly."""
import numpy as np
import pytest
import torch

from gpu_common import dm, np_, say

pytestmark = pytest.mark.gpu


def lists(X, Y, K):
    d = np.zeros((len(X), len(Y)), np.float32)
    for k in range(X.shape[1]):   # one rounding per term: the FP64 product and sum of FP32 values, rounded
        e = (X[:, k, None] - Y[None, :, k]).astype(np.float64)
        d = (e * e + d).astype(np.float32)
    return (np.argsort(d, 1, kind="stable")[:, :K], np.argsort(d.T, 1, kind="stable")[:, :K])


@pytest.mark.parametrize("nx,ny,D,K", [(1, 1, 1, 1), (63, 65, 31, 5), (64, 64, 32, 64), (129, 100, 33, 100),
                                       (40, 2048, 8, 7), (40, 2049, 8, 7), (300, 70, 130, 48), (200, 200, 3, 17)])
@pytest.mark.parametrize("ties", [False, True])
def test_fp32_lists_are_exact(nx, ny, D, K, ties):
    rng = np.random.default_rng([nx, ny, D])
    # small whole numbers: exact distances, most of them tied
    draw = (lambda n: rng.integers(-1, 2, (n, D))) if ties else (lambda n: rng.integers(-2**10, 2**10, (n, D)))
    X, Y = draw(nx).astype(np.float32), draw(ny).astype(np.float32)
    if not ties and D > 8:
        X, Y = X / 1024, Y / 1024   # products of 22 bits: the FP64 sum before rounding is exact
    K = min(K, nx, ny)
    say(f"  {nx} x {ny} x {D}, K={K}")
    want = lists(X, Y, K)
    ctx = dm().Context(0)
    for call in (ctx.knn_candidates, ctx.knn_candidates_noalloc):
        got = call(torch.from_numpy(X), torch.from_numpy(Y), K, "fp32")
        assert all(np.array_equal(np_(g), w) for g, w in zip(got, want))
    if ties:   # BF16 holds these values, and FP32 their sums, exactly
        got = ctx.knn_candidates(torch.from_numpy(X), torch.from_numpy(Y), K, "bf16")
        assert all(np.array_equal(np_(g), w) for g, w in zip(got, want))


def test_a_refused_call_leaves_the_outputs_alone():
    ctx = dm().Context(0)
    X, Y = torch.randn(50, 16), torch.randn(60, 16)
    X[49, 15] = float("inf")
    out = (torch.full((50, 4), -7, dtype=torch.int32, device="cuda"),
           torch.full((60, 4), -7, dtype=torch.int32, device="cuda"))
    with pytest.raises(dm().DMError) as e:
        ctx.knn_candidates_noalloc(X, Y, 4, "bf16", out=out)
    torch.cuda.synchronize()
    assert e.value.code == -5 and all(bool((o == -7).all()) for o in out)
