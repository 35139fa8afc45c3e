"""The search of short rows in one launch behind the first pass: rows on their prediction, rows without one, the whole
general search, each with the blocks of a row waiting for one another and with waits that run out, in any order."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS

WAIT = 1 << 16                                                  # longer than any wait by default
# (mode of the search, bound of its waits): after a wait that ran out the next search finds its histograms not zero
STEPS = [(None, WAIT), (0, WAIT), (1, 0), (1, WAIT), (4, 3), (0, WAIT), (4, WAIT), (1, 2), (0, 0), (0, WAIT), (4, 0), (1, WAIT)]


# rows of one block (16 tiles), of two, of many; too many rows for more than one block each; a list longer than one block
# takes (uniform magnitudes crowd the band); the two random-k draws in one set of launches, with k and bands of their own
@pytest.mark.parametrize("wc,sc,N,d,wk,sk,uniform", [
    ("topk", "topk", 2, 16_384, 300, 700, False), ("topk", "topk", 2, 16_385, 300, 700, False),
    ("topk", "topk", 3, 70_001, 4000, 1000, False), ("topk", "topk", 1, 1_000_003, 60_000, 40_000, True),
    ("topk", "identity", 140, 20_001, 200, 0, False), ("topk", "topk", 33, 40_000, 999, 999, False),
    ("randk", "randk", 3, 70_001, 4000, 70, False), ("randk", "randk", 140, 20_001, 200, 90, False),
    ("randk", "randk", 2, 1_000_003, 500, 600, False), ("randk", "topk", 5, 33_333, 333, 33, False),
    ("identity", "randk", 2, 50_000, 0, 512, False)])
def test_search_modes_and_waits_in_any_order(wc, sc, N, d, wk, sk, uniform):
    say(f"case short rows {wc}/{sc} N={N} d={d} k={wk}/{sk}")
    import oracle
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(d + N)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, wc, sc, wk, sk, 0.05) as ctx:
        ctx.set_random(7, 0)
        for t, (mode, wait) in enumerate(STEPS):
            g = rng.standard_normal((N, d), dtype=np.float32)
            if uniform:
                g = (0.5 + rng.random((N, d), dtype=np.float32) * np.float32(0.4 if t % 2 else 0.5)).astype(np.float32)
            if mode is not None:
                ctx.force_search_mode(mode)
            ctx.set_search_wait(wait)
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            torch.cuda.synchronize()
            oracle.step(g, x, e, wc, sc, 0.05, wk, sk, rng=(7, t))
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}: mode {mode}, wait {wait}"
            if mode == 4:
                assert ctx.info().slow_rows == (N if wk else 0) + (1 if sk else 0), f"step {t}"


def test_a_search_that_one_block_repeated_is_reported():
    """Rows without a prediction are listed by the blocks that share them; when their waits run out block 0 searches the whole
    row, which counts as a general search."""
    say("case report of searches whose waits ran out")
    from paper_2402_11857_amd import LiecContext

    N, d, k = 3, 70_001, 700
    g = torch.randn((N, d), dtype=torch.float32, device=DEV)
    x, e = torch.zeros_like(g), torch.zeros(d, dtype=torch.float32, device=DEV)
    with LiecContext(N, d, "topk", "topk", k, k, 0.05) as ctx:
        for wait in (WAIT, 0, WAIT):
            ctx.force_search_mode(1)
            ctx.set_search_wait(wait)
            ctx.step(g, x, e)
            assert ctx.info().slow_rows == (0 if wait else N + 1), wait
            for row in range(N + 1):
                st = ctx.search_state(row)
                assert (st["general_search"], st["listed"] > 0) == ((0, True) if wait else (1, False)), (wait, row, st)
            ctx.set_search_wait(WAIT)
            ctx.step(g, x, e)                                   # on the band that either search predicts
            assert ctx.info().slow_rows == 0


@pytest.mark.parametrize("N,d", [(1, 16_384), (129, 5), (129, 1024), (140, 17_001), (300, 3000)])
def test_rows_that_one_block_searches_are_listed_like_any_other(N, d):
    """Short rows and many rows: one block a row.  Without a prediction it makes the first digit's list and the candidate
    bitmap (ties and zeros among the values: the bin of one key, the bin of zeros)."""
    say(f"case rows of one block N={N} d={d}")
    import oracle
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(d)
    k = max(1, d // 50)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, "topk", "topk", k, k, 0.05) as ctx:
        for t, mode in enumerate([None, 1, 0, 4, 1]):
            g = rng.standard_normal((N, d), dtype=np.float32)
            if t == 4:
                g = np.where(rng.random((N, d)) < 0.3, np.round(g * 4) / 4, 0).astype(np.float32)
            if mode is not None:
                ctx.force_search_mode(mode)
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            torch.cuda.synchronize()
            oracle.step(g, x, e, "topk", "topk", 0.05, k, k)
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"
            assert ctx.info().slow_rows == (N + 1 if mode == 4 else 0), f"step {t}"
