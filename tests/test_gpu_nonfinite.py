"""Inf and NaN among the inputs: what reaches the models, and what liec_get_info reports."""
import numpy as np
import pytest
import torch

from _gpu import DEV, GPU_MARKS, say
import oracle
from paper_2402_11857_amd import LiecContext

pytestmark = GPU_MARKS

INF, NAN = float("inf"), float("nan")


def same(a, b):
    """Bit for bit, any NaN equal to any other (which of two NaN operands an operation hands on is not specified)."""
    return np.array_equal(np.where(np.isnan(a), np.uint32(1), a.view(np.uint32)),
                          np.where(np.isnan(b), np.uint32(1), b.view(np.uint32)))


def state(N, d, seed):
    rng = np.random.default_rng(seed)
    g = rng.standard_normal((N, d)).astype(np.float32)
    return g, rng.standard_normal((N, d)).astype(np.float32), rng.standard_normal(d).astype(np.float32)


@pytest.mark.parametrize("sc", ["identity", "sign", "blocksign", "topk", "randk"])
@pytest.mark.parametrize("N,d", [(1, 5), (3, 1024), (5, 70_001)])
@pytest.mark.parametrize("bad", [(INF,), (NAN,), (INF, -INF)])
def test_an_uncompressed_gradient_that_is_not_finite_reaches_its_workers_model(sc, N, d, bad):
    """g - p^i is Inf - Inf = NaN there and +0 for the other workers, whatever the server sends of the column."""
    say(f"case non-finite identity/{sc} N={N} d={d} {bad}")
    g, x, e = state(N, d, d + N)
    for j in (0, d // 2, d - 1):                                # the last one: the end of a row off a 16-byte boundary
        for i, value in enumerate(bad):
            g[(N - 1 + i) % N, j] = value
    k, off = max(1, d // 100), [0, 2, d]
    dev = [torch.from_numpy(a.copy()).to(DEV) for a in (g, x, e)]
    with LiecContext(N, d, "identity", sc, 0, k, 0.1) as ctx:
        if sc == "blocksign":
            ctx.set_blocks(off)
        ctx.set_random(3, 0)
        ctx.step(*dev)
        torch.cuda.synchronize()
    oracle.step_blocks(g, x, e, "identity", sc, 0.1, off, 0, k, rng=(3, 0))
    assert np.isnan(x).any() and same(dev[1].cpu().numpy(), x), "models"
    assert same(dev[2].cpu().numpy(), e), "server error"
