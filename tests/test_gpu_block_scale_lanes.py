"""Blockwise workers: a wave of the aggregation, by tile or by chunk, loads the scales of 64 rows at a time, a lane each."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


@pytest.mark.parametrize("d", [2048 * 1024 + 3, 20_003])
@pytest.mark.parametrize("N,sc", [(63, "blocksign"), (65, "sign"), (73, "blocksign"), (3, "identity")])
def test_scales_of_more_rows_than_lanes(N, sc, d):
    """The kernel by tile runs from 2048 tiles of 1024 columns on; a boundary inside a tile and one between tiles."""
    import oracle
    from paper_2402_11857_amd import LiecContext

    say(f"case block scales by lane N={N} d={d} server {sc}")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(N)
    g = torch.empty((N, d), device=DEV).normal_(generator=gen).mul_(torch.arange(1, N + 1, device=DEV)[:, None])   # every row a scale of its own
    x = torch.zeros((N, d), device=DEV)
    e = torch.empty(d, device=DEV).normal_(generator=gen)
    off = [0, 5 * 1024, d // 3, d]
    xo, eo = np.zeros((N, d), dtype=np.float32), e.cpu().numpy()
    with LiecContext(N, d, "blocksign", sc, 0, 0, 0.1) as ctx:
        ctx.set_blocks(off)
        ctx.step(g, x, e)
        oracle.step_blocks(g.cpu().numpy(), xo, eo, "blocksign", sc, 0.1, off)
        assert H.bit_equal(e.cpu().numpy(), eo)
        assert H.bit_equal(x.cpu().numpy(), xo)
