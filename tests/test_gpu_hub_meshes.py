"""Product spaces of meshes with hub vertices, which neighbour every other one: the
closedness rows' sort keys number a vertex's neighbours, so those of a hub need
many (compact keys), or too many for 32 bits (wide keys).  Bit for bit against the
oracle."""
import numpy as np
import pytest

from gpu_common import dm, say
from oracle import oracle as O
from test_gpu_space import _compare_space

pytestmark = pytest.mark.gpu


def bipyramid(n, hubs_last):
    """Two apexes over a ring of n vertices; the apexes first or last."""
    a = 2 * np.pi * np.arange(n) / n
    ring = np.stack([np.cos(a), np.sin(a), 0.1 * np.sin(3 * a)], 1)
    apex = np.array([[0, 0, 1.0], [0, 0, -1.0]])
    i, j = np.arange(n), np.roll(np.arange(n), -1)
    up, down, shift = (n, n + 1, 0) if hubs_last else (0, 1, 2)
    V = np.concatenate([ring, apex] if hubs_last else [apex, ring])
    F = np.concatenate([np.stack([np.full(n, up), i + shift, j + shift], 1),
                        np.stack([np.full(n, down), j + shift, i + shift], 1)])
    return V.astype(np.float32), F.astype(np.int32)


def lists(n, m, K, hubs_last, other_last):
    """K candidates of every vertex: those around its place on the other ring; of an
    apex, the apexes and the first of the ring."""
    apexes, first = ([m, m + 1], 0) if other_last else ([0, 1], 2)
    at = (np.arange(n) * m // n)[:, None] + np.arange(K)[None] - K // 2
    ring = at % m + first
    apex = np.tile(np.concatenate([apexes, np.arange(K - 2) + first]), (2, 1))
    return np.concatenate([ring, apex] if hubs_last else [apex, ring]).astype(np.int32)


@pytest.mark.parametrize("nx,ny,K", [(4, 5, 4), (40, 33, 9), (250, 250, 8), (1200, 900, 6)])   # the last: wide keys
@pytest.mark.parametrize("hubs_last", [False, True])
def test_hub_space_matches_the_oracle(nx, ny, K, hubs_last):
    VX, FX = bipyramid(nx, hubs_last)
    VY, FY = bipyramid(ny, not hubs_last)
    cxy, cyx = lists(nx, ny, K, hubs_last, not hubs_last), lists(ny, nx, K, not hubs_last, hubs_last)
    S = O.Space(VX, FX, VY, FY, cxy, cyx)
    ctx = dm().Context(0)
    ctx.build_product_space(VX, FX, VY, FY, cxy, cyx)
    say(f"  {nx} and {ny} on the rings: {ctx.info['n_prod_tri']} elements, {ctx.info['n_rows_full']} rows, {ctx.info['n_cand']} pairs")
    _compare_space(S, ctx)
