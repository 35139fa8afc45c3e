"""Scaled sign on both sides, rows of middling length: partial sums of 16-wave blocks, finished by the kernels that use them."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


# either side of 2048, 4096 and 8192 wave tiles in all, remainders of a block's 16 tiles, 8 workers and more, none left over
@pytest.mark.parametrize("N,d,own", [(16, 131_073, False), (3, 699_400, False), (3, 700_001, False), (1, 2_097_153, False),
                                     (9, 262_144 + 5, False), (4, 1_048_576, False), (4, 1_048_577, False), (5, 1_000_003, False),
                                     (16, 524_288, False), (16, 524_289, True)])
def test_partial_sums_of_wide_blocks(N, d, own):
    say(f"case wide sums N={N} d={d}")
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(N + d)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, "sign", "sign", 0, 0, 0.05) as ctx:
        for t in range(2):
            g = rng.standard_normal((N, d), dtype=np.float32)
            ctx.profile_begin(1)
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            assert ("worker_l1_final" in ctx.profile_end()) == own
            info, desc = ctx.info(), ctx.worker_desc()
            wdesc, sdesc = H.oracle_step_rows(g, x, e, "sign", "sign", 0.05)[:2]
            # fp64 sums of d terms in another order: at most d units of 2^-53 apart, far less than an fp32 scale resolves
            assert all(abs(a - w.l1) <= d * 2.0 ** -53 * w.l1 for a, w in zip(desc["l1"], wdesc))
            assert desc["scale"] == [float(np.float32(w.scale)) for w in wdesc] and info.server_scale == np.float32(sdesc.scale)
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"


@pytest.mark.parametrize("N,tiles,extra,wide", [(2, 2048, 0, True), (2, 2064, 1, False), (1, 2065, 0, False), (5, 1632, 0, True),
                                                (5, 1633, 0, False), (16, 512, 0, True)])
def test_wide_blocks_only_where_the_aggregation_takes_the_sums(N, tiles, extra, wide):
    """Rows of up to 129 sums, up to 512 in all: beyond, narrow blocks and a kernel that finishes the sums are faster."""
    say(f"case wide blocks N={N} tiles={tiles}+{extra}")
    import oracle
    from paper_2402_11857_amd import LiecContext

    d = tiles * 1024 + extra
    g = np.random.default_rng(tiles).standard_normal((N, d), dtype=np.float32)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.zeros((N, d), dtype=torch.float32, device=DEV), torch.zeros(d, dtype=torch.float32, device=DEV)
    with LiecContext(N, d, "sign", "sign", 0, 0, 0.1) as ctx:
        ctx.profile_begin(1)
        ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
        assert ("worker_l1_final" in ctx.profile_end()) == (not wide)
    oracle.step(g, x, e, "sign", "sign", 0.1)
    assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e)
