"""The scratch that liec_create takes stays within what the header states."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(__file__))
from _gpu import GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


# per row, in KiB: short list 128 (one launch, up to 128 workers) or 32; digit histograms of a row with several blocks 23, one of
# its share of a list for each block (64 at most); first-digit histogram 16 where a side takes several launches
@pytest.mark.parametrize("wc,sc", [("topk", "topk"), ("randk", "randk"), ("topk", "identity"), ("randk", "topk")])
@pytest.mark.parametrize("N,d,k,per_row", [(1, 5_000_000, 50, 231), (3, 2_000_000, 20, 216), (4, 40_000_000, 200, 230), (128, 40_000, 40, 156),
                                           (129, 40_000, 40, 33), (300, 2000, 20, 33), (5000, 100, 2, 33)])
def test_scratch_is_what_the_header_says(wc, sc, N, d, k, per_row):
    say(f"case scratch {wc}/{sc} N={N} d={d}")
    from paper_2402_11857_amd import LiecContext

    tiles = -(-d // 1024)                                       # v and the bitmaps cover whole tiles of 1024 columns
    bound = 4096 * tiles + (N + 1) * 8 * (min(d // 16, 8 * k) + 4097)
    bound += (N + 1) * tiles * 128 if "randk" in (wc, sc) else 0
    bound += (N if wc == "topk" else 0) * tiles * 32 + (tiles * 32 if sc == "topk" else 0)
    bound += 8 * (N * -(-tiles // 4) + tiles)                   # partial sums of either side
    bound += 256 * (N + 1) + 64                                 # descriptors
    with LiecContext(N, d, wc, sc, k, k, 0.1) as ctx:
        left = (ctx.scratch_bytes() - bound) / (N + 1) / 1024
    assert left <= per_row <= 232, f"{left:.1f} KiB a row of histograms and short lists"
