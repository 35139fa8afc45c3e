"""The aggregation's forms (a wave per chunk of 256 columns, a wave per tile of 1024) around the sizes where they
split the work: batches of 8 rows, ends of chunks and tiles, and rows on the far side of the rule that picks a form.
"""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


def _chain(N, d, wc, sc, k, steps, off=None, batching=None):
    import oracle
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(N * 1000 + d)
    x = rng.standard_normal((N, d), dtype=np.float32)
    e = np.float32(0.1) * rng.standard_normal(d, dtype=np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, wc, sc, k, k, 0.05) as ctx:
        if off is not None:
            ctx.set_blocks(off)
        ctx.set_random(9, 0)
        for t in range(steps):
            if batching is not None:
                ctx.set_gather_batching((t + batching) % 2)
            g = rng.standard_normal((N, d), dtype=np.float32)
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            torch.cuda.synchronize()
            if off is not None:
                oracle.step_blocks(g, x, e, wc, sc, 0.05, off)
            else:
                H.oracle_step_rows(g, x, e, wc, sc, 0.05, k, k, rng=(9, t))
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"


@pytest.mark.parametrize("wc,sc", [("topk", "sign"), ("topk", "blocksign"), ("randk", "sign"), ("identity", "sign"),
                                   ("identity", "topk"), ("blocksign", "blocksign"), ("sign", "sign"),
                                   ("topk", "topk"), ("randk", "topk"), ("blocksign", "topk")])
@pytest.mark.parametrize("N,d", [(1, 1024), (7, 1025), (8, 255), (9, 257), (16, 1280), (17, 3079)])
def test_aggregate_small(N, d, wc, sc):
    say(f"case aggregate N={N} d={d} {wc}/{sc}")
    off = None
    if "blocksign" in (wc, sc):
        off = [0, 3, 254, d] if d > 254 else [0, 3, d]          # boundaries inside a group of 4 columns and near a chunk's end
    if off is not None and "topk" in (wc, sc):
        _chain_blocks_topk(N, d, off, wc, sc)
    else:
        _chain(N, d, wc, sc, max(1, d // 10), 3, off, 0 if wc == "topk" else None)


def _chain_blocks_topk(N, d, off, wc, sc):
    import oracle
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(d)
    k = max(1, d // 10)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, wc, sc, k, k, 0.05) as ctx:
        ctx.set_blocks(off)
        for t in range(3):
            g = rng.standard_normal((N, d), dtype=np.float32)
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            torch.cuda.synchronize()
            oracle.step_blocks(g, x, e, wc, sc, 0.05, off, k, k)
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"


# first lengths (and one more tile) that take a wave per tile
@pytest.mark.parametrize("wc,sc,N,d", [("topk", "sign", 2, 8192 * 1024 + 5), ("topk", "sign", 2, 8191 * 1024),
                                       ("randk", "sign", 2, 8192 * 1024 + 1028), ("randk", "sign", 64, 255 * 1024), ("blocksign", "sign", 3, 2048 * 1024 + 7),
                                       ("blocksign", "sign", 3, 2047 * 1024),
                                       # the aggregation makes a top-k server's first filter pass, and does not any more
                                       ("topk", "topk", 2, 4096 * 1024), ("topk", "topk", 2, 4096 * 1024 + 3),
                                       ("identity", "topk", 2, 4095 * 1024 + 6), ("identity", "topk", 2, 4096 * 1024 + 4)])
def test_aggregate_either_side_of_the_rule(wc, sc, N, d):
    say(f"case aggregate rule N={N} d={d} {wc}/{sc}")
    off = [0, 5, d // 3 + 2, d // 3 + 3, d - 1, d] if wc == "blocksign" else None
    _chain(N, d, wc, sc, d // 500, 3 if sc == "topk" else 2, off)


# a wave per tile: batches of 16 rows, lists from a few entries to more than they hold, columns that several or all
# workers keep, both forms of the candidate bitmap, and rows that have none
@pytest.mark.parametrize("N", [1, 15, 16, 17, 33])
@pytest.mark.parametrize("d,k", [(1024, 1), (1024, 1000), (1025, 60), (5000, 40), (5003, 1500), (30_001, 300)])
@pytest.mark.parametrize("same", [0.0, 0.5, 1.0])
def test_aggregate_by_tile(N, d, k, same):
    say(f"case aggregate by tile N={N} d={d} k={k} same={same}")
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(N * 7 + d + k)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, "topk", "sign", k, 0, 0.05) as ctx:
        ctx.set_gather_batching(0)
        for t in range(4):
            g = rng.standard_normal((N, d), dtype=np.float32)
            common = rng.random(d) < same                       # columns whose gradient all workers share, up to the scale
            g[:, common] = (g[0, common] * (1.0 + 0.001 * np.arange(N)[:, None])).astype(np.float32)
            ctx.set_group_bitmap(t % 2)
            if t == 3:
                ctx.force_search_mode(4)                        # no valid bitmap: every column is a candidate
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            torch.cuda.synchronize()
            H.oracle_step_rows(g, x, e, "topk", "sign", 0.05, k, 0)
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"


# a chunk per wave: up to 4 rows take a kernel that asks for 4 rows' words; both forms of the candidate bitmap, rows that have none
@pytest.mark.parametrize("sc", ["sign", "topk", "identity"])
@pytest.mark.parametrize("N,d,k", [(1, 1021, 30), (2, 5000, 40), (3, 5003, 1500), (4, 1028, 60), (5, 1025, 1000)])
def test_aggregate_few_rows_by_chunk(N, d, k, sc):
    say(f"case aggregate few rows N={N} d={d} k={k} server {sc}")
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(N * 7 + d + k)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, "topk", sc, k, k, 0.05) as ctx:
        for t in range(4):
            g = rng.standard_normal((N, d), dtype=np.float32)
            ctx.set_group_bitmap(t % 2)
            if t == 3:
                ctx.force_search_mode(4)                        # no valid bitmap: every column is a candidate
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            torch.cuda.synchronize()
            H.oracle_step_rows(g, x, e, "topk", sc, 0.05, k, k)
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"


@pytest.mark.parametrize("N,d,k", [(64, 256 * 1024, 300), (64, 256 * 1024 + 3, 200_000), (70, 240 * 1024, 20_000)])
def test_aggregate_by_tile_randk(N, d, k):
    say(f"case aggregate by tile randk N={N} d={d} k={k}")
    _chain(N, d, "randk", "sign", k, 2)


# a blockwise server's partial sums, left by the aggregation or, on tables with many boundaries in one 4096-column tile,
# by the pass over v: rounds with waves beyond the last tile, blocks that end with a tile
@pytest.mark.parametrize("wc", ["sign", "blocksign"])
@pytest.mark.parametrize("N,d", [(2, 1), (3, 1025), (9, 4096), (2, 4097), (5, 12_289), (2, 70_001), (2, 2048 * 1024 + 1030)])
@pytest.mark.parametrize("table", ["one", "tiles", "crowded"])
def test_blockwise_sums_by_tile(wc, N, d, table):
    say(f"case blockwise sums N={N} d={d} {wc} {table}")
    off = {"one": [0, d], "tiles": list(range(0, d, 4096)) + [d],
           "crowded": sorted({0, 1, 2, 5, 1023, 1024, 1500, 4095, d // 2, d // 2 + 1, d - 1, d} - {o for o in range(d + 1, 4097)})}[table]
    off = [o for o in sorted(set(off)) if 0 <= o <= d]
    _chain(N, d, wc, "blocksign", 1, 2, off)


# as many items in a tile as the aggregation sums itself (3 on the shortest rows, 5 at a million columns, never more
# than 8), one more, and as many as a tile has columns: the pass over v sums those
@pytest.mark.parametrize("wc", ["sign", "blocksign"])
@pytest.mark.parametrize("N,d,items,by_pass", [(2, 9_000, 3, False), (2, 9_000, 4, True), (2, 1024 * 1024 + 2, 5, False),
                                               (2, 1024 * 1024 + 2, 6, True), (1, 4096 * 1024 + 1, 8, False),
                                               (1, 4096 * 1024 + 1, 9, True), (3, 8195, 4096, True)])
def test_blockwise_sums_of_a_crowded_tile(wc, N, d, items, by_pass):
    say(f"case blockwise sums of a crowded tile N={N} d={d} {wc} items={items}")
    from paper_2402_11857_amd import LiecContext

    off = list(range(4096, 4096 + items)) + [8192, d]           # the second tile: one-column blocks and the rest of it
    off = [0] + off
    _chain(N, d, wc, "blocksign", 1, 2, off)
    g, x, e = (torch.ones(s, device=DEV) for s in ((N, d), (N, d), d))
    with LiecContext(N, d, wc, "blocksign", 0, 0, 0.05) as ctx:
        ctx.set_blocks(off)
        ctx.profile_begin(1)
        ctx.step(g, x, e)
        short = wc == "blocksign" and d < 2048 * 1024           # (a wave per chunk leaves no sums)
        assert ("server_l1" in ctx.profile_end()) == (by_pass or short)


# a wave per tile: as many flagged groups of 4 columns as are listed (48 a row in the fine bitmap, 12 lines in the coarse
# one, 512 in all), one fewer and one more, on rows that keep one column of each of their first groups and little else
@pytest.mark.parametrize("N,groups", [(1, 48), (2, 96), (10, 480), (11, 512), (16, 512), (17, 512)])
@pytest.mark.parametrize("extra", [-1, 0, 1])
@pytest.mark.parametrize("coarse", [0, 1])
def test_aggregate_at_the_limit_of_the_list(N, groups, extra, coarse):
    say(f"case aggregate list limit N={N} flagged={groups + extra} coarse={coarse}")
    from paper_2402_11857_amd import LiecContext

    rows = min(N, 16)
    flagged = (min(12 * rows, groups) if coarse else groups) + extra     # of the first 16 rows
    width = 16 if coarse else 4
    d, k = 2048, -(-flagged // rows)                            # every row keeps k columns
    rng = np.random.default_rng(N + groups + extra)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, "topk", "sign", k, 0, 0.05) as ctx:
        ctx.set_gather_batching(0)
        ctx.set_group_bitmap(coarse)
        for t in range(3):
            g = np.float32(1e-6) * rng.standard_normal((N, d), dtype=np.float32)
            for i in range(N):
                mine = flagged // rows + (1 if i % 16 < flagged % rows else 0)
                at = np.arange(k) * width + rng.integers(0, width, k)
                at[mine:] = (at[0] // 4 * 4 + np.arange(4))[at[0] // 4 * 4 + np.arange(4) != at[0]][:k - mine]   # (in a flagged group)
                g[i, at] = rng.uniform(1.0, 1.001, k)
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            torch.cuda.synchronize()
            H.oracle_step_rows(g, x, e, "topk", "sign", 0.05, k, 0)
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"


# the aggregation sums three items in every tile: boundaries inside a group of 4 columns, at a wave's end, next to a tile's end
@pytest.mark.parametrize("wc,N,d", [("sign", 3, 12_289), ("sign", 17, 70_001), ("blocksign", 2, 2048 * 1024 + 1030)])
def test_blockwise_sums_at_block_boundaries(wc, N, d):
    say(f"case blockwise sums at boundaries N={N} d={d} {wc}")
    from paper_2402_11857_amd import LiecContext

    off = [0]
    for t in range(0, d, 4096):
        off += [o for o in (t + (1024 if t // 4096 % 2 else 1501), t + (4094 if t // 4096 % 3 else 4095)) if o < d]
    off.append(d)
    _chain(N, d, wc, "blocksign", 1, 2, off)
    with LiecContext(N, d, wc, "blocksign", 0, 0, 0.05) as ctx:
        ctx.set_blocks(off)
        ctx.profile_begin(1)
        ctx.step(*(torch.ones(s, device=DEV) for s in ((N, d), (N, d), d)))
        assert "server_l1" not in ctx.profile_end()
