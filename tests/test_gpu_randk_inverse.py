"""Random-k on thin bands, where the priorities above the band are walked and inverted instead of hashing every column:
the ends of the walk (bands from a few words to many blocks of 2^16), columns at the row's end, few and many rows."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


@pytest.mark.parametrize("N,d,k", [(2, 400_001, 1), (1, 655_360, 9), (3, 700_003, 3), (2, 1_048_577, 64), (9, 1_310_721, 90),
                                   (2, 3_000_001, 800), (1, 6_000_000, 4_000)])
@pytest.mark.parametrize("seed", [0, 0xFFFF_FFFF_FFFF_FFFF])
def test_thin_bands(N, d, k, seed):
    say(f"case randk inverse N={N} d={d} k={k} seed={seed}")
    import oracle
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(d)
    g = rng.standard_normal((N, d), dtype=np.float32)
    gd = torch.from_numpy(g).to(DEV)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    idx, val = torch.empty(k, dtype=torch.int32, device=DEV), torch.empty(k, device=DEV)
    with LiecContext(N, d, "randk", "randk", k, k, 0.05) as ctx:
        ctx.set_random(seed, 5)
        for t in range(2):
            ctx.step(gd, xd, ed)
            torch.cuda.synchronize()
            H.oracle_step_rows(g, x, e, "randk", "randk", 0.05, k, k, rng=(seed, 5 + t))
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"
        for i in range(N):
            ctx.pack_topk_message(gd, i, idx, val)
            torch.cuda.synchronize()
            ri, rv = oracle.pack_randk(g[i], k, rng=(seed, 6, i))
            assert np.array_equal(idx.cpu().numpy().view(np.uint32), ri) and H.bit_equal(val.cpu().numpy(), rv)
