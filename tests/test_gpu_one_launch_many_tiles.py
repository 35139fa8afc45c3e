"""The search in one launch on more than 32768 tiles of 1024 columns in all: rows that several blocks share, rows of one block each."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


@pytest.mark.parametrize("N,d,k", [(34, 1_000_001, 3000), (2100, 16_001, 40)])
def test_rows_in_every_mode(N, d, k):
    """No prediction, a prediction, none again with waits that run out, the whole general search."""
    say(f"case one launch on many tiles N={N} d={d}")
    import oracle
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(N)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, "topk", "sign", k, 0, 0.05) as ctx:
        for t, (mode, wait) in enumerate([(None, 1 << 16), (None, 1 << 16), (1, 0), (4, 1 << 16)]):
            g = rng.standard_normal((N, d), dtype=np.float32)
            if mode is not None:
                ctx.force_search_mode(mode)
            ctx.set_search_wait(wait)
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            torch.cuda.synchronize()
            oracle.step(g, x, e, "topk", "sign", 0.05, k, 0)
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}: mode {mode}, wait {wait}"
        # one launch: the slots of the several launches do not appear
        ctx.set_search_wait(1 << 16)
        ctx.profile_begin(1)
        ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
        assert "worker_hist0" not in ctx.profile_end()
