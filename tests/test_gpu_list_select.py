"""The end of the threshold search: few entries compared with one another, many entries of one key ordered by index."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


def _row(rng, d, above, ties, spread):
    """`above` entries over 1, `ties` entries of magnitude 1 (either sign) at random places, the rest below 1;
    spread: how far the others lie from 1 (small: many of them fall into the predicted band)."""
    v = (1.0 - spread * rng.random(d)).astype(np.float32)
    v[v >= 1.0] = np.float32(1.0) - np.float32(spread)
    at = rng.permutation(d)
    v[at[:above]] = (1.0 + spread * (0.01 + rng.random(above))).astype(np.float32)
    v[at[above:above + ties]] = 1.0
    return v * rng.choice(np.array([-1.0, 1.0], np.float32), d)


# counts around the 256 bins of a digit, beyond one index digit's bin, and all of a narrow band
@pytest.mark.parametrize("d", [200_000, 199_997])
@pytest.mark.parametrize("ties,where", [(1, "only"), (2, "last"), (255, "middle"), (256, "first"), (257, "middle"), (257, "last"),
                                        (300, "first"), (4095, "middle"), (4097, "last"), (9000, "middle")])
@pytest.mark.parametrize("spread", [0.9, 0.02])
def test_ties_at_the_threshold(d, ties, where, spread):
    say(f"case list select d={d} ties={ties} {where} spread={spread}")
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(ties * 7 + d)
    N, above = 2, 2000
    k = above + {"only": 1, "first": 1, "middle": (ties + 1) // 2, "last": ties}[where]
    g = np.stack([_row(rng, d, above, ties, spread) for _ in range(N)])
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    gd = torch.from_numpy(g).to(DEV)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, "topk", "sign", k, 0, 0.05) as ctx:
        for t in range(3):                                      # first-digit band, then predicted bands
            ctx.step(gd, xd, ed)
            torch.cuda.synchronize()
            wdesc = H.oracle_step_rows(g, x, e, "topk", "sign", 0.05, k, 0)[0]
            got = ctx.worker_desc()
            assert got["tau_key"] == [w.tau_key for w in wdesc] and got["cutoff"] == [w.cutoff for w in wdesc], f"step {t}"
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"


# lists either side of the 16384 entries one block holds: uniform keys, so that the first band is crowded
@pytest.mark.parametrize("k", [1000, 20_000, 60_000])
def test_list_lengths(k):
    say(f"case list select lengths k={k}")
    from paper_2402_11857_amd import LiecContext

    N, d = 2, 1_000_003
    rng = np.random.default_rng(k)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, "topk", "topk", k, k, 0.05) as ctx:
        for t in range(4):
            g = (0.5 + rng.random((N, d), dtype=np.float32) * np.float32(0.4 if t % 2 else 0.5)).astype(np.float32)
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            torch.cuda.synchronize()
            H.oracle_step_rows(g, x, e, "topk", "topk", 0.05, k, k)
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"
