"""Scaled sign on short rows, where the aggregation and the update form the scales from the partial sums themselves:
either side of the rules that pick this, and the scales the caller can query."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


# few and many workers' partial sums (the rule's edges: below); the server's: 2048 blocks of the update and above
@pytest.mark.parametrize("wc", ["sign", "identity", "topk", "randk", "blocksign"])
@pytest.mark.parametrize("N,d", [(1, 1), (3, 4097), (64, 32_768), (64, 32_769), (65, 4_100), (32, 65_536), (33, 65_536), (1, 262_144),
                                 (1, 262_145), (1, 1_048_577), (2, 1_048_580)])
def test_scales_formed_by_their_users(N, d, wc):
    say(f"case folded scales N={N} d={d} {wc}")
    import oracle
    from paper_2402_11857_amd import LiecContext

    if wc == "blocksign" and d < 2:
        pytest.skip("fewer columns than blocks")
    rng = np.random.default_rng(N + d)
    off = [0, d // 2, d]
    k = max(1, d // 100)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, wc, "sign", k, 0, 0.05) as ctx:
        if wc == "blocksign":
            ctx.set_blocks(off)
        ctx.set_random(3, 0)
        for t in range(2):
            g = rng.standard_normal((N, d), dtype=np.float32)
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            info, desc = ctx.info(), ctx.worker_desc()
            if wc == "blocksign":
                oracle.step_blocks(g, x, e, wc, "sign", 0.05, off)
            else:
                wdesc, sdesc = H.oracle_step_rows(g, x, e, wc, "sign", 0.05, k, 0, rng=(3, t))[:2]
                assert info.server_scale == np.float32(sdesc.scale) and abs(info.server_l1 - sdesc.l1) <= 1e-12 * sdesc.l1
                if wc == "sign":
                    assert desc["scale"] == [float(np.float32(w.scale)) for w in wdesc]
            assert info.nonfinite == 0
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"
        g[N - 1, d // 2] = np.inf
        ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
        if wc != "randk":                                       # a draw does not look at the gradients and may leave it out
            assert ctx.info_status()[0].nonfinite == 1


# the aggregation forms the scales of up to 16 workers and 512 partial sums; a kernel of its own does beyond that
@pytest.mark.parametrize("N,d,own_kernel", [(16, 4_097, False), (17, 4_097, True), (64, 1_000, True), (16, 131_072, False),
                                            (16, 131_073, True), (1, 2_097_152, False), (1, 2_097_153, True)])
def test_which_kernel_forms_the_workers_scales(N, d, own_kernel):
    say(f"case who forms the scales N={N} d={d}")
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(N + d)
    g = rng.standard_normal((N, d), dtype=np.float32)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    with LiecContext(N, d, "sign", "identity", 0, 0, 0.05) as ctx:
        ctx.profile_begin(1)
        ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
        assert ("worker_l1_final" in ctx.profile_end()) == own_kernel
        wdesc = H.oracle_step_rows(g, x, e, "sign", "identity", 0.05)[0]
        assert ctx.worker_desc()["scale"] == [float(np.float32(w.scale)) for w in wdesc]
    assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e)
