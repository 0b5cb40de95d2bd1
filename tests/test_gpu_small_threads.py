"""The one-workgroup sweep from two threads at once, each with its own context,
stream and problem size: what a launch may ask of the LDS is a setting of the
kernel, so a small problem's call must not lower it under a larger one's.
Results are those of the same calls one after the other, bit for bit."""
import threading

import pytest
import torch

from gpu_common import dm, say
from test_gpu_row_forms import rows_of_one_shape

pytestmark = pytest.mark.gpu

SIZES = {"fp64": ((3, 3, 560), (3, 3, 420)), "fp32": ((3, 3, 690), (8, 8, 300))}   # 50 to 100 KB of state


def solver(shape, prec):
    n, ptr, cols, coefs, rhs, cost = rows_of_one_shape(*shape, 0, 4)
    ctx = dm().Context(0)
    ctx.build_ilp(n, ptr, cols, coefs, rhs)
    ctx.set_costs(torch.from_numpy(cost))
    say(f"  {shape} {prec}: {ctx.info['nnz']} nonzeros, {ctx.info['n_free']} variables")
    return ctx


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_two_sizes_on_two_threads(prec):
    ctxs = [solver(s, prec) for s in SIZES[prec]]
    want = [c.dual_solve(c.init_lambda(prec), 3)[0].clone() for c in ctxs]
    torch.cuda.synchronize()
    bad = []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(100):
                    got, _ = ctxs[i].dual_solve(ctxs[i].init_lambda(prec), 3)
                    if not torch.equal(got, want[i]):
                        bad.append(i)
                torch.cuda.current_stream().synchronize()
        except Exception as e:   # a thread's exception would pass unseen
            bad.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad[:3]
