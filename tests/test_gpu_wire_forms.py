"""The message kernels around the sizes where they split the work: words of a sign message at any byte, the counts and
positions of kept entries over tiles and blocks, candidate bitmaps of either form and rows without one.
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


# lengths around a byte, a 32-column word, the 8 lanes a thread packs, a chunk and a tile
@pytest.mark.parametrize("d", [1, 7, 9, 31, 33, 63, 255, 257, 1023, 1025, 4101])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_sign_bits_at_any_byte(d, offset):
    say(f"case sign bits d={d} offset={offset}")
    import oracle
    from paper_2402_11857_amd import LiecContext

    N = 2
    g = np.random.default_rng(d).standard_normal((N, d)).astype(np.float32)
    nb = (d + 7) // 8
    x, e = torch.zeros((N, d), device=DEV), torch.zeros(d, device=DEV)
    flat = torch.full((16 + nb + 16,), 0xA5, dtype=torch.uint8, device=DEV)
    out = flat[8 + offset:8 + offset + nb]
    p = torch.full((d + 64,), 7.0, device=DEV)
    with LiecContext(N, d, "sign", "sign", 0, 0, 0.1) as ctx:
        ctx.step(torch.from_numpy(g).to(DEV), x, e)
        scales = ctx.worker_desc()["scale"]
        for i in range(N):
            ctx.pack_sign_bits(i, out)
            ctx.unpack_sign_message(out, [scales[i]], False, p[offset:offset + d])
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), oracle.pack_sign(g[i]))
            assert H.bit_equal(p[offset:offset + d].cpu().numpy(), oracle.compress("sign", g[i])[0])
            ph = p.cpu().numpy()
            assert np.all(ph[:offset] == 7.0) and np.all(ph[offset + d:] == 7.0)
    h = flat.cpu().numpy()
    assert np.all(h[:8 + offset] == 0xA5) and np.all(h[8 + offset + nb:] == 0xA5)


def _check(ctx, comp, g, k, i, rng, gd):
    import oracle

    N, d = g.shape
    idx = torch.full((k,), -1, dtype=torch.int32, device=DEV)
    val = torch.zeros(k, device=DEV)
    p = torch.full((d,), 3.0, device=DEV)
    ctx.pack_topk_message(gd, i, idx, val)
    ctx.unpack_topk_message(idx, val, p)
    torch.cuda.synchronize()
    if comp == "topk":
        ri, rv = oracle.pack_topk(g[i], k)
        ref = oracle.compress("topk", g[i], k)[0]
    else:
        ri, rv = oracle.pack_randk(g[i], k, rng=(rng[0], rng[1], i))
        ref = oracle.compress("randk", g[i], k, rng=(rng[0], rng[1], i))[0]
    assert np.array_equal(idx.cpu().numpy().view(np.uint32), ri), f"worker {i}: indices"
    assert H.bit_equal(val.cpu().numpy(), rv), f"worker {i}: values"
    assert H.bit_equal(p.cpu().numpy(), ref), f"worker {i}: decompressed"


# one tile, one block of 4 tiles and the next one, blocks beyond 1024 and beyond 4096 counts, and rows whose blocks own more
# than 4 tiles
@pytest.mark.parametrize("comp", ["topk", "randk"])
@pytest.mark.parametrize("N,d,k", [(2, 1, 1), (2, 1000, 1000), (3, 4096, 40), (2, 4097, 4000), (2, 70_003, 3500),
                                   (2, 4_300_001, 20_000), (1, 16_780_300, 10_000), (1, 33_600_001, 50_000)])
def test_kept_entries(comp, N, d, k):
    say(f"case kept entries {comp} N={N} d={d} k={k}")
    from paper_2402_11857_amd import LiecContext

    g = np.random.default_rng(d + k).standard_normal((N, d), dtype=np.float32)
    gd = torch.from_numpy(g).to(DEV)
    x, e = torch.zeros((N, d), device=DEV), torch.zeros(d, device=DEV)
    with LiecContext(N, d, comp, "sign", k, 0, 0.1) as ctx:
        ctx.set_random(31, 4)
        for t in range(2):                                      # without a prediction, then with one
            if comp == "topk":
                ctx.set_group_bitmap(t)
            ctx.step(gd, x, e)
            if comp == "topk":
                ctx.set_group_bitmap(1 - t)                     # what the next step will write, not what this one wrote
            for i in range(N if t else 1):
                _check(ctx, comp, g, k, i, (31, 4 + t), gd)


@pytest.mark.parametrize("comp", ["topk", "randk"])
def test_kept_entries_of_rows_without_a_bitmap(comp):
    say(f"case kept entries general search {comp}")
    from paper_2402_11857_amd import LiecContext

    N, d, k = 2, 50_001, 6000
    g = np.random.default_rng(3).standard_normal((N, d)).astype(np.float32)
    g[:, 100:] = np.float32(0.5)                                # far more equal magnitudes than a list holds
    gd = torch.from_numpy(g).to(DEV)
    x, e = torch.zeros((N, d), device=DEV), torch.zeros(d, device=DEV)
    with LiecContext(N, d, comp, "sign", k, 0, 0.1) as ctx:
        ctx.set_random(8, 0)
        ctx.force_search_mode(4)
        ctx.step(gd, x, e)
        assert ctx.info().slow_rows == N
        for i in range(N):
            _check(ctx, comp, g, k, i, (8, 0), gd)


def test_kept_entries_of_a_constant_row():
    """No bitmap, the kept entries all at the row's start: the blocks of the rest look at their tiles' counts only."""
    say("case kept entries constant row")
    from paper_2402_11857_amd import LiecContext

    N, d, k = 1, 4_200_003, 30_000
    g = np.full((N, d), 0.5, np.float32)
    g[0, 1_500_000] = 2.0                                       # and one more, far from them
    gd = torch.from_numpy(g).to(DEV)
    x, e = torch.zeros((N, d), device=DEV), torch.zeros(d, device=DEV)
    with LiecContext(N, d, "topk", "sign", k, 0, 0.1) as ctx:
        for t in range(2):
            ctx.step(gd, x, e)
            assert ctx.info().slow_rows == N
            _check(ctx, "topk", g, k, 0, None, gd)


@pytest.mark.parametrize("captured", [0, 1])
def test_kept_entries_after_a_replayed_step(captured):
    """The bitmap a message is packed from is in the form of the step that ran last, also when that was the replay of a
    captured one and a step in the other form was called in between."""
    say(f"case kept entries after a replay, captured form {captured}")
    from paper_2402_11857_amd import LiecContext

    N, d, k = 3, 70_003, 700
    rng = np.random.default_rng(captured)
    gs = [rng.standard_normal((N, d), dtype=np.float32) for _ in range(4)]
    g, x, e = torch.zeros((N, d), device=DEV), torch.zeros((N, d), device=DEV), torch.zeros(d, device=DEV)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with LiecContext(N, d, "topk", "sign", k, 0, 0.1, stream=s) as ctx, torch.cuda.stream(s):
        def step(data, form):
            g.copy_(torch.from_numpy(data))
            ctx.set_group_bitmap(form)
            ctx.step(g, x, e)
            for i in range(N):
                _check(ctx, "topk", data, k, i, None, g)

        step(gs[0], captured)
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        graph.capture_begin()
        ctx.step(g, x, e)
        graph.capture_end()
        for t in range(1, 4):
            step(gs[0], 1 - captured)
            g.copy_(torch.from_numpy(gs[t]))
            graph.replay()
            for i in range(N):
                _check(ctx, "topk", gs[t], k, i, None, g)
        s.synchronize()
        del graph
