"""Candidates where memory holds the distances once but not twice: the call
does without their transpose, and its lists are the same."""
import pytest
import torch

from gpu_common import dm, say

pytestmark = pytest.mark.gpu


def test_distances_fit_once_but_not_twice():
    n, K = 20000, 3
    one = 4 * n * n   # bytes of the distances
    g = torch.Generator(device="cuda").manual_seed(1)
    # whole numbers, whose squared distances are exact in FP32
    X, Y = (torch.randint(-1024, 1024, (n, 3), generator=g, device="cuda").float() for _ in range(2))
    ctx = dm().Context(0)
    want = [c.clone() for c in ctx.knn_candidates(X, Y, K, "fp32")]
    torch.cuda.synchronize()
    ctx.close()   # gives its memory back
    ctx = dm().Context(0)
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    held = torch.empty(free - one * 3 // 2, dtype=torch.uint8, device="cuda")
    say(f"  {free / 1e9:.1f} GB free, {torch.cuda.mem_get_info()[0] / 1e9:.2f} left for {one / 1e9:.2f} of distances")
    try:
        got = ctx.knn_candidates(X, Y, K, "fp32")
        torch.cuda.synchronize()
    finally:
        del held
        torch.cuda.empty_cache()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    # and against the distances themselves, for some of the rows
    for c, P, Q in ((got[0], X, Y), (got[1], Y, X)):
        d = ((P[:200, None] - Q[None]) ** 2).sum(2).long()
        key = d * n + torch.arange(n, device="cuda")   # ties to the lower index
        assert torch.equal(key.topk(K, dim=1, largest=False, sorted=True).indices.int(), c[:200])
