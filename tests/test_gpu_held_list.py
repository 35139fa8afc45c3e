"""Lists one block selects from: lengths at which the passes over them take another form or another round."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


def _check(N, d, n, levels):
    """n values in [1, 1.0625), which share their first digit, the others below 1/4; with levels, of so many magnitudes only."""
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(n + levels)
    k = (n + 1) // 2
    g = (0.25 * rng.random((N, d))).astype(np.float32)
    for row in g:
        top = rng.random(n) if not levels else rng.integers(0, levels, n) / levels
        row[rng.permutation(d)[:n]] = (1.0 + 0.0624 * top).astype(np.float32)
    keys = g.view(np.uint32).copy()
    g *= rng.choice(np.array([-1.0, 1.0], np.float32), (N, d))
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    gd, xd, ed = torch.from_numpy(g).to(DEV), torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, "topk", "sign", k, 0, 0.05) as ctx:
        for t in range(3):                                      # the digit's bin, then predicted bands
            before = [ctx.search_state(i) for i in range(N)]
            ctx.step(gd, xd, ed)
            torch.cuda.synchronize()
            wdesc = H.oracle_step_rows(g, x, e, "topk", "sign", 0.05, k, 0)[0]
            got = ctx.worker_desc()
            assert got["tau_key"] == [w.tau_key for w in wdesc] and got["cutoff"] == [w.cutoff for w in wdesc], f"step {t}"
            for i in range(N):                                  # every row's list was the one that the step began with
                st, want = ctx.search_state(i), n
                if t > 0:
                    want = int(((keys[i] >= before[i]["lo"]) & (keys[i] < before[i]["hi"])).sum())
                    assert before[i]["mode"] == 0 and st["misses"] == 0
                assert (st["listed"], st["general_search"]) == (want, 0), f"step {t} row {i}"
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"
        ctx.profile_begin(1)
        ctx.step(gd, xd, ed)
        return ctx.profile_end()


# up to 128 entries are compared without a digit, 1024 threads walk the list, 2048 entries are one load each, 12288 the most that leave all
# copies of the bins their place, 16384 the most that are held
@pytest.mark.parametrize("levels", [0, 3])
@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 1023, 1025, 2048, 2049, 8193, 12287, 12288, 12289, 16383, 16384, 16385])
def test_list_of_n_entries(n, levels):
    say(f"case held list n={n} levels={levels}")
    assert "worker_hist0" not in _check(2, 300_007, n, levels)  # one launch


# one key that more entries share than are held
def test_list_of_one_key_beyond_what_is_held():
    say("case list of one key, 22000 entries")
    assert "worker_hist0" not in _check(2, 300_007, 22_000, 1)


# the same where several launches search: rows of more than 8192 tiles
@pytest.mark.parametrize("n,levels", [(128, 0), (129, 0), (2049, 3), (12288, 0), (12289, 3), (16384, 3), (16385, 0),
                                      (40_000, 0), (40_000, 1), (300_000, 0), (300_001, 3), (300_000, 1500)])
def test_list_of_n_entries_on_a_long_row(n, levels):
    say(f"case held list, long row, n={n} levels={levels}")
    assert "worker_hist0" in _check(1, 8192 * 1024 + 5, n, levels)
