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


# up to 128 entries are compared without a digit, 1024 threads walk the list, 2048 entries are one load each, 12288 the most that are held
@pytest.mark.parametrize("levels", [0, 3])
@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 1023, 1025, 2048, 2049, 8193, 12287, 12288, 12289, 16385])
def test_list_of_n_entries(n, levels):
    """n values in [1, 1.0625), which share their first digit, the others below 1/4; with levels, of so many magnitudes only."""
    say(f"case held list n={n} levels={levels}")
    from paper_2402_11857_amd import LiecContext

    N, d = 2, 300_007
    rng = np.random.default_rng(n + levels)
    k = (n + 1) // 2
    g = (0.25 * rng.random((N, d))).astype(np.float32)
    for row in g:
        top = rng.random(n) if not levels else rng.integers(0, levels, n) / levels
        row[rng.permutation(d)[:n]] = (1.0 + 0.0624 * top).astype(np.float32)
    g *= rng.choice(np.array([-1.0, 1.0], np.float32), (N, d))
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    gd, xd, ed = torch.from_numpy(g).to(DEV), torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, "topk", "sign", k, 0, 0.05) as ctx:
        for t in range(3):                                      # the digit's bin, then predicted bands
            ctx.step(gd, xd, ed)
            torch.cuda.synchronize()
            wdesc = H.oracle_step_rows(g, x, e, "topk", "sign", 0.05, k, 0)[0]
            got = ctx.worker_desc()
            assert got["tau_key"] == [w.tau_key for w in wdesc] and got["cutoff"] == [w.cutoff for w in wdesc], f"step {t}"
            if t == 0:
                assert ctx.search_state(0)["listed"] in (n, 0)  # (0: more than the list holds)
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"
