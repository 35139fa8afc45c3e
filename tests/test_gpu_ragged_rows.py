"""Rows that do not start at multiples of 16 bytes: every kernel's 128-bit accesses at any 4-byte address, the
element-wise end of a row, and nothing touched outside the caller's buffers.
"""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
import _harness as H  # noqa: E402
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS

GUARD = 64                    # sentinel values on either side of a buffer
SENTINEL = np.float32(-123.456)


class Guarded:
    """A contiguous device tensor that starts `offset` floats past a 256-byte boundary, with sentinels around it."""

    def __init__(self, host: np.ndarray, offset: int):
        self.flat = torch.full((GUARD + 64 + host.size + GUARD,), float(SENTINEL), dtype=torch.float32, device=DEV)
        self.at = GUARD + offset
        self.t = self.flat[self.at:self.at + host.size].view(host.shape)
        self.t.copy_(torch.from_numpy(host))

    def untouched_outside(self) -> bool:
        h = self.flat.cpu().numpy()
        return bool(np.all(h[:self.at] == SENTINEL) and np.all(h[self.at + self.t.numel():] == SENTINEL))


def _case(N, d, seed):
    rng = np.random.default_rng(seed)
    g = rng.standard_normal((N, d)).astype(np.float32)
    x = rng.standard_normal((N, d)).astype(np.float32)
    e = (0.1 * rng.standard_normal(d)).astype(np.float32)
    return g, x, e


PAIRS = [("sign", "sign"), ("topk", "topk"), ("topk", "sign"), ("identity", "identity"), ("randk", "randk"),
         ("blocksign", "blocksign")]


# the lengths around a group of 4 columns, a chunk of 256, a tile of 1024 and a block of 4096; offsets that put the
# rows of g, x and e at different places inside a 16-byte group
@pytest.mark.parametrize("wc,sc", PAIRS)
@pytest.mark.parametrize("N,d,offsets", [(3, 1, (1, 2, 3)), (2, 2, (0, 0, 0)), (3, 3, (3, 1, 0)), (2, 4, (1, 1, 1)),
                                         (3, 5, (0, 0, 0)), (2, 7, (2, 0, 1)), (3, 257, (0, 3, 0)), (2, 1022, (1, 0, 2)),
                                         (3, 1023, (0, 0, 0)), (2, 1027, (2, 2, 2)), (3, 4097, (0, 1, 3)),
                                         (2, 8192, (1, 2, 3)), (2, 70_001, (3, 3, 1))])
def test_ragged_rows_step(N, d, offsets, wc, sc):
    say(f"case ragged N={N} d={d} offsets={offsets} {wc}/{sc}")
    import oracle
    from paper_2402_11857_amd import LiecContext

    if wc == "blocksign" and d < 3:
        pytest.skip("fewer columns than blocks")
    g, x, e = _case(N, d, N * 1000 + d)
    k = max(1, d // 50)
    off = [0, 1, max(2, d // 2), d] if d >= 4 else [0, 1, d]
    gd, xd, ed = (Guarded(a, o) for a, o in zip((g, x, e), offsets))
    with LiecContext(N, d, wc, sc, k, k, 0.05) as ctx:
        if wc == "blocksign":
            ctx.set_blocks(off)
        ctx.set_random(5, 0)
        for t in range(3):                                     # no prediction, then predicted bands
            ctx.step(gd.t, xd.t, ed.t)
            torch.cuda.synchronize()
            if wc == "blocksign":
                oracle.step_blocks(g, x, e, wc, sc, 0.05, off)
            else:
                oracle.step(g, x, e, wc, sc, 0.05, k, k, rng=(5, t))
            assert H.bit_equal(xd.t.cpu().numpy(), x) and H.bit_equal(ed.t.cpu().numpy(), e), f"step {t}"
        ctx.step_sync(gd.t, xd.t, ed.t)
        torch.cuda.synchronize()
        oracle.step_sync(g, x, e, 0.05)
        assert H.bit_equal(xd.t.cpu().numpy(), x) and H.bit_equal(ed.t.cpu().numpy(), e), "averaging iteration"
    assert gd.untouched_outside() and xd.untouched_outside() and ed.untouched_outside()
    assert H.bit_equal(gd.t.cpu().numpy(), g)
