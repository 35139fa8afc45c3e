"""The search on more than 32768 tiles of 1024 columns in all: one launch for very many short rows, several for the others."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


@pytest.mark.parametrize("N,d,k,one", [(34, 1_000_001, 3000, False), (2100, 16_001, 40, True)])
def test_rows_in_every_mode(N, d, k, one):
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
        # the slots of the several launches appear, or not.  (With few blocks a row, one row that misses its band would hold up a single launch)
        ctx.set_search_wait(1 << 16)
        ctx.profile_begin(1)
        ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
        assert ("worker_hist0" not in ctx.profile_end()) == one


@pytest.mark.parametrize("N,d,one", [(512, 131_071, True), (512, 131_073, False), (511, 131_071, False), (64, 524_288, True),
                                     (64, 524_289, False)])
def test_where_one_launch_ends(N, d, one):
    """512 rows are two rounds of the chip's 256 compute units, 131072 columns 128 tiles, 64 x 524288 columns 32768."""
    say(f"case one launch N={N} d={d}")
    from paper_2402_11857_amd import LiecContext

    gen = torch.Generator(device=DEV)
    gen.manual_seed(N)
    g = torch.empty((N, d), device=DEV).normal_(generator=gen)
    x, e = torch.zeros((N, d), device=DEV), torch.zeros(d, device=DEV)
    with LiecContext(N, d, "topk", "sign", d // 100, 0, 0.05) as ctx:
        ctx.profile_begin(1)
        ctx.step(g, x, e)
        assert ("worker_hist0" not in ctx.profile_end()) == one
