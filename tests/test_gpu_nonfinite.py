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


@pytest.mark.parametrize("wc,where", [("identity", "g"), ("identity", "e"), ("blocksign", "e"), ("topk", "e"), ("randk", "e")])
@pytest.mark.parametrize("N,d", [(3, 65_536), (2, 70_001)])
@pytest.mark.parametrize("bad", [INF, NAN])
def test_a_top_k_server_that_filters_v_where_it_is_formed_reports_it(wc, where, N, d, bad):
    """Short rows, a server row on its predicted band: the aggregation is the only kernel that looks at v."""
    say(f"case non-finite report {wc}/topk N={N} d={d} {where} {bad}")
    g, x, e = (torch.from_numpy(a).to(DEV) for a in state(N, d, d + N))
    k = d // 100
    with LiecContext(N, d, wc, "topk", k, k, 0.1) as ctx:
        if wc == "blocksign":
            ctx.set_blocks([0, 5, d // 2, d])
        for t in range(3):
            e.copy_(torch.from_numpy(state(N, d, d + N)[2]))    # the same v each step: the server's prediction holds
            ctx.set_random(1, 0)
            ctx.step(g, x, e)
        info, status = ctx.info_status()
        assert status == 0 and info.nonfinite == 0
        misses = info.band_misses
        e.copy_(torch.from_numpy(state(N, d, d + N)[2]))
        (g[N - 1] if where == "g" else e)[d - 1] = bad
        ctx.set_random(1, 0)
        ctx.profile_begin(1)
        ctx.step(g, x, e)
        assert "server_filter_warm" not in ctx.profile_end()    # (the aggregation made that pass)
        info, status = ctx.info_status()
        assert status == 4 and info.nonfinite == 1
        assert info.band_misses == misses and ctx.search_state(N)["general_search"] == 0
        e.copy_(torch.from_numpy(state(N, d, d + N)[2]))
        g[N - 1, d - 1] = 0.5
        ctx.step(g, x, e)
        assert ctx.info_status()[1] == 0                        # and a step later it is gone
