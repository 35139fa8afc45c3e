"""The two predictions of a row's threshold: the trend where it drifts, the last value where it goes up and down."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


@pytest.mark.parametrize("kind", ["alternating", "drifting", "jumps of a bf16 step"])
def test_band_follows_the_thresholds(kind):
    say(f"case band prediction, {kind}")
    import oracle
    from paper_2402_11857_amd import LiecContext

    N, d, k, steps = 1, 60_000, 900, 40
    rng = np.random.default_rng(5)
    base = rng.standard_normal((N, d), dtype=np.float32)
    if kind == "jumps of a bf16 step":
        base = (base.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
    x, e = np.zeros((N, d), np.float32), np.zeros(d, np.float32)
    xd, ed = torch.from_numpy(x).to(DEV), torch.from_numpy(e).to(DEV)
    taus, widths, early = [], [], 0
    with LiecContext(N, d, "topk", "sign", k, 0, 0.05) as ctx:
        for t in range(steps):
            if kind == "alternating":
                g = base * np.float32(1.0 + 0.02 * (t & 1))
            elif kind == "drifting":
                g = base * np.float32(1.005 ** t)
            else:                                               # one bf16 step up after every ninth step
                g = (base.view(np.uint32) + np.uint32((t // 10) << 16)).view(np.float32)
            ctx.step(torch.from_numpy(g).to(DEV), xd, ed)
            torch.cuda.synchronize()
            oracle.step(g, x, e, "topk", "sign", 0.05, k, 0)
            assert H.bit_equal(xd.cpu().numpy(), x) and H.bit_equal(ed.cpu().numpy(), e), f"step {t}"
            st = ctx.search_state(0)
            taus.append(ctx.worker_desc()["tau_key"][0])
            widths.append(st["hi"] - st["lo"])
            if t == 12:
                early = ctx.info().band_misses
        late = ctx.info().band_misses - early
    change = max(abs(a - b) for a, b in zip(taus[1:], taus)) if kind != "drifting" else abs(taus[-1] - taus[-2])
    assert late == 0, "no prediction may fail once the changes are known"
    if kind == "alternating":                                   # six times the change on either side, not twelve
        assert widths[-1] <= 2 * 6 * change + 2 * (1 << 15), (widths[-1], change)
    elif kind == "drifting":                                    # the trend: a few changes wide, or the floor
        assert widths[-1] <= max(2 * 4 * change, 2 << 15), (widths[-1], change)
