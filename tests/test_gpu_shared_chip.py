"""Two contexts whose searches each spread over most of the chip, stepping at the same time on two streams: blocks of either
may be resident in part and wait for the rest.  Every wait is bounded, and a search whose wait ran out is done by one block."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


@pytest.mark.parametrize("mode", [1, 4])
@pytest.mark.parametrize("sizes", [((8, 300_000), (8, 300_000)), ((2, 1_100_003), (40, 65_536))])
def test_searches_without_a_prediction_on_two_streams(sizes, mode):
    say(f"case shared chip {sizes} mode {mode}")
    import oracle
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(3)
    streams = [torch.cuda.Stream() for _ in sizes]
    gs = [rng.standard_normal((N, d), dtype=np.float32) for N, d in sizes]
    gd = [torch.from_numpy(g).to(DEV) for g in gs]
    xd = [torch.zeros_like(g) for g in gd]
    ed = [torch.zeros(d, dtype=torch.float32, device=DEV) for _, d in sizes]
    torch.cuda.synchronize()
    ctx = [LiecContext(N, d, "topk", "topk", d // 100, d // 50, 0.1, stream=s) for (N, d), s in zip(sizes, streams)]
    steps = 4
    for _ in range(steps):
        for c in ctx:
            c.force_search_mode(mode)
        for c, g, x, e in zip(ctx, gd, xd, ed):
            c.step(g, x, e)
    for c, s in zip(ctx, streams):
        s.synchronize()
        c.close()
    for (N, d), g, x, e in zip(sizes, gs, xd, ed):
        xo, eo = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
        for _ in range(steps):
            oracle.step(g, xo, eo, "topk", "topk", 0.1, d // 100, d // 50)
        assert H.bit_equal(x.cpu().numpy(), xo) and H.bit_equal(e.cpu().numpy(), eo)
