"""Decompression of sign messages on either side of the length from which its threads loop over smaller blocks."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(__file__))
from _gpu import DEV, GPU_MARKS, say  # noqa: E402

pytestmark = GPU_MARKS


@pytest.mark.parametrize("blockwise", [False, True])
@pytest.mark.parametrize("d", [1, 1023, 4097, 16_777_215, 16_777_216, 16_777_217, 16_777_221])
def test_dense_message(d, blockwise):
    say(f"case unpack blocks d={d} blockwise={blockwise}")
    from paper_2402_11857_amd import LiecContext

    rng = np.random.default_rng(d)
    bits = rng.integers(0, 256, (d + 7) // 8, dtype=np.uint8)
    off = sorted({0, d // 3, d // 2 + 1, d}) if d > 3 else [0, d]
    scales = [0.25 * (b + 1) for b in range(len(off) - 1)] if blockwise else [0.75]
    s = np.repeat(np.float32(scales), np.diff(off)) if blockwise else np.float32(scales[0])
    want = np.where(np.unpackbits(bits, count=d, bitorder="little"), -s, s).astype(np.float32)
    with LiecContext(1, d, "sign", "sign", 0, 0, 0.1) as ctx:
        if blockwise:
            ctx.set_blocks(off)
        p = torch.full((d,), 7.0, device=DEV)
        ctx.unpack_sign_message(torch.from_numpy(bits).to(DEV), scales, blockwise, p)
        assert np.array_equal(p.cpu().numpy(), want)
