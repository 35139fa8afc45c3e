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


# rows from 28672 tiles on (the last one cut off): the scales of 64 rows at a time
LONG = 28_672 * 1024 - 5


@pytest.mark.parametrize("sc", ["sign", "blocksign"])
def test_long_rows(sc):
    import oracle
    from paper_2402_11857_amd import LiecContext

    say(f"case block scales by lane, long rows, server {sc}")
    N, d = 3, LONG
    gen = torch.Generator(device=DEV)
    gen.manual_seed(4)
    g = torch.empty((N, d), device=DEV).normal_(generator=gen).mul_(torch.arange(1, N + 1, device=DEV)[:, None])
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


def test_long_rows_more_than_lanes():
    """65 rows against the same operations in torch: with e = x = 0 every fused multiply-add is a single rounded product."""
    from paper_2402_11857_amd import LiecContext

    say("case block scales by lane, 65 long rows")
    N, d, lr = 65, LONG, 0.25
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    g = torch.empty((N, d), device=DEV)
    for i in range(N):
        g[i].normal_(generator=gen).mul_(i + 1)
    x, e = torch.zeros((N, d), device=DEV), torch.zeros(d, device=DEV)
    off = [0, 5 * 1024, d // 3, d]
    with LiecContext(N, d, "blocksign", "identity", 0, 0, lr) as ctx:
        ctx.set_blocks(off)
        ctx.step(g, x, e)
        scales = torch.tensor(ctx.block_scales()[0], dtype=torch.float32, device=DEV).reshape(N, len(off) - 1)
    sizes = torch.tensor(np.diff(off), device=DEV)

    def message(i):
        s = torch.repeat_interleave(scales[i], sizes, output_size=d)
        return torch.where(g[i] < 0, -s, s)

    acc = torch.zeros(d, device=DEV)
    for i in range(N):
        acc += message(i)
    p = acc * torch.tensor(np.float32(1) / np.float32(N), device=DEV)
    assert not bool(e.any())
    for i in range(N):
        assert torch.equal(x[i], (p + (g[i] - message(i))) * -lr), f"row {i}"
