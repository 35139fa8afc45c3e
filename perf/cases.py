"""What the speed of this framework is measured on: calls a training program makes through `LiecContext`.

A compressed iteration (`step`) for each operator that is used in earnest, the averaging iteration (`step_sync`), and the
wire forms of the messages (`pack_*` / `unpack_*`), from the smallest simulated model to the largest that this
repository is configured for, rows that are a multiple of four long and rows that are not.  Inputs are seeded: per-layer
Gaussian gradients, heavy-tailed outliers or bf16 mantissas where a case says so, models that start out equal on all
workers, a server error that is not zero.  A state carries two gradient batches that the passes take in turn, as a
training loop hands a new batch to every step.
"""
from __future__ import annotations

import math

import torch

from paper_2402_11857_amd import LiecContext

LAYERS = 32                  # parameter tensors a row is made of, each with a gradient scale of its own
BATCHES = 2                  # gradient batches of a state

# sizes of one simulated worker's model: ResNet-18, ResNet-50 and VGG-16 (as in workloads/layers.py)
R18, R50, VGG = 11_689_512, 25_557_032, 138_357_544

PAIRS = (("sign", "sign"), ("blocksign", "blocksign"), ("topk", "topk"), ("topk", "sign"), ("randk", "randk"),
         ("identity", "identity"))


def _case(what, worker, server, N, d, k=0, blocks=0, lr=0.1, outliers=False, bf16=False, **kw):
    return dict(kw, what=what, worker=worker, server=server, N=N, d=d, k=k, blocks=blocks, lr=lr, outliers=outliers, bf16=bf16)


def listed():
    return [
        # the smallest simulation: a step of a few microseconds' work, so what counts is launches and latency
        _case("step", "sign", "sign", 4, 65_536, name="sign_tiny"),
        # a mid-sized layer group under top-k: caches hold it, many short dependent kernels
        _case("step", "topk", "topk", 8, 1_048_576, k=10_485, lr=0.05, name="topk_mid"),
        # a small top-k run on a model whose length is odd, gradients from a bf16 backward pass (many ties)
        _case("step", "topk", "topk", 5, 3_000_017, k=30_000, bf16=True, name="topk_ragged_bf16"),
        # the paper's operator, blockwise scaled sign with 14 blocks, odd row length and odd number of workers
        _case("step", "blocksign", "blocksign", 7, 7_340_033, blocks=14, name="blocksign_ragged"),
        # the ordinary scaled-sign step: 16 workers of a ResNet-18-sized model
        _case("step", "sign", "sign", 16, R18, outliers=True, name="sign_r18"),
        # the uncompressed baseline (identity on both sides is parallel SGD) that every experiment runs beside it;
        # a classification head of another width makes the row length even but not a multiple of four
        _case("step", "identity", "identity", 8, R18 + 2, name="psgd_ragged"),
        # many workers, sparse messages both ways: a ResNet-50-sized model
        _case("step", "topk", "topk", 32, R50, k=R50 // 1000, outliers=True, name="topk_r50"),
        # the same with random-k
        _case("step", "randk", "randk", 32, R50, k=R50 // 1000, name="randk_r50"),
        # the largest: 16 workers of a VGG-16-sized model, top-k up, scaled sign down
        _case("step", "topk", "sign", 16, VGG, k=VGG // 200, lr=0.01, name="mixed_vgg"),
        # the averaging iteration that every 32nd or 100th step is
        _case("average", "sign", "sign", 16, R18, name="average_r18"),
        # exchange of scaled-sign messages: every worker's wire bits packed, every message unpacked
        _case("wire", "sign", "sign", 8, R18 + 1, name="wire_sign_ragged"),
        # exchange of top-k messages as (index, value) pairs
        _case("wire", "topk", "topk", 8, R18, k=R18 // 100, name="wire_topk"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """1 to 64 workers, rows of 2^16 to 1.4e8 columns (any remainder by four), at most 4e8 elements, k/d from 0.05 % to 5 %."""
    what = rng.choice(("step",) * 5 + ("average", "wire"))
    worker, server = rng.choice(PAIRS)
    if what == "wire":
        worker = server = rng.choice(("sign", "topk", "randk"))
    N = _log_uniform(rng, 1, 64 if what != "wire" else 16)
    d = _log_uniform(rng, 65_536, min(VGG, 400_000_000 // N if what != "wire" else 200_000_000 // N))
    if rng.random() < 0.5:
        d -= d % 4
    k = max(1, int(d * math.exp(rng.uniform(math.log(5e-4), math.log(5e-2))))) if {worker, server} & {"topk", "randk"} else 0
    blocks = rng.randint(2, 64) if worker == "blocksign" else 0
    return _case(what, worker, server, N, d, k=k, blocks=blocks, lr=rng.choice((0.01, 0.05, 0.1)),
                 outliers=rng.random() < 0.4, bf16=rng.random() < 0.2)


# ---- inputs ------------------------------------------------------------------------------------------------------
def _offsets(case):
    """Block table: uneven blocks of whole columns."""
    B, d = case["blocks"], case["d"]
    return [d * b // B + (b % 3) for b in range(B)] + [d] if B else None


def _inputs(case, seed, batches):
    """(gradient batches, x, server error, seed of the random-k draws)"""
    N, d = case["N"], case["d"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    scale = 10.0 ** (3.0 * torch.rand(LAYERS, generator=gen, device="cuda") - 4.0)        # 1e-4 .. 1e-1
    sizes = torch.tensor([d * (i + 1) // LAYERS - d * i // LAYERS for i in range(LAYERS)], device="cuda")
    sigma = torch.repeat_interleave(scale, sizes, output_size=d)
    grads = []
    for _ in range(batches):
        g = torch.empty((N, d), dtype=torch.float32, device="cuda")
        for i in range(N):
            row = g[i].normal_(generator=gen)
            if case["outliers"]:                            # one element in a thousand from a Student-t with 2 degrees
                pick = torch.rand(d, generator=gen, device="cuda") < 1e-3
                u = torch.rand(d, generator=gen, device="cuda").clamp_(min=1e-30)
                z = torch.randn(d, generator=gen, device="cuda")
                row.copy_(torch.where(pick, z / torch.sqrt(-torch.log(u)), row))
            row.mul_(sigma)
            if case["bf16"]:
                row.copy_(row.bfloat16())
        grads.append(g)
    x = torch.empty((N, d), dtype=torch.float32, device="cuda")
    x[0].normal_(0.0, 0.02, generator=gen)
    x[1:] = x[0]
    e = torch.empty(d, dtype=torch.float32, device="cuda").normal_(generator=gen).mul_(sigma)
    return grads, x, e, seed * 2 + 1


def _context(case, rng_seed):
    ctx = LiecContext(case["N"], case["d"], case["worker"], case["server"], case["k"], case["k"], case["lr"])
    if case["blocks"]:
        ctx.set_blocks(_offsets(case))
    ctx.set_random(rng_seed, 0)
    return ctx


def prepare(case, seed):
    wire = case["what"] == "wire"
    grads, x, e, rng_seed = _inputs(case, seed, 1 if wire else BATCHES)
    state = dict(case=case, ctx=_context(case, rng_seed), grads=grads, x=x, e=e, t=0)
    if wire:
        N, d, k = case["N"], case["d"], case["k"]
        state["ctx"].step(grads[0], x, e)                   # the step whose messages are exchanged
        state["p"] = torch.empty((N, d), dtype=torch.float32, device="cuda")
        if case["worker"] == "sign":
            state["bits"] = torch.empty((N, (d + 7) // 8), dtype=torch.uint8, device="cuda")
            state["scales"] = state["ctx"].worker_desc()["scale"]
        else:
            state["idx"] = torch.empty((N, k), dtype=torch.int32, device="cuda")
            state["val"] = torch.empty((N, k), dtype=torch.float32, device="cuda")
    return state


def run(state):
    case, ctx = state["case"], state["ctx"]
    if case["what"] == "wire":
        p = state["p"]
        if case["worker"] == "sign":
            for i in range(case["N"]):
                ctx.pack_sign_bits(i, state["bits"][i])
            for i in range(case["N"]):
                ctx.unpack_sign_message(state["bits"][i], state["scales"][i:i + 1], False, p[i])
            return state["bits"], p
        for i in range(case["N"]):
            ctx.pack_topk_message(state["grads"][0], i, state["idx"][i], state["val"][i])
        for i in range(case["N"]):
            ctx.unpack_topk_message(state["idx"][i], state["val"][i], p[i])
        return state["idx"], state["val"], p
    g = state["grads"][state["t"] % BATCHES]
    state["t"] += 1
    if case["what"] == "average":
        ctx.step_sync(g, state["x"], state["e"])
    else:
        ctx.step(g, state["x"], state["e"])
    return state["x"], state["e"]


def work(case):
    N, d, k = case["N"], case["d"], case["k"]
    if case["what"] == "wire":
        if case["worker"] == "sign":                        # bits out, bits in, dense message out
            return {"bytes": N * (3 * (d // 8) + 4 * d), "flops": N * d}
        return {"bytes": N * (4 * d + 16 * k + 4 * d), "flops": N * d}
    # gradients and models read, models written; the server error read and written
    return {"bytes": 12 * N * d + 8 * d, "flops": 6 * N * d}


def tolerance(case):
    # include/liec.h states every rounding and the order of every fp32 sum (worker order, then one fused multiply-add);
    # only the fp64 sum behind a scale is free in its order, and that leaves the rounded fp32 scale as it is
    return "exact"


# ---- the same in 64 bits -------------------------------------------------------------------------------------------
def _top(key, k):
    """Mask of the k largest keys, equal ones to the lower index."""
    mask = torch.zeros(key.numel(), dtype=torch.bool, device=key.device)
    mask[torch.sort(key, descending=True, stable=True)[1][:k]] = True
    return mask


_M64 = (1 << 64) - 1


def _mix(z):
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9 & _M64
    z = (z ^ (z >> 27)) * 0x94D049BB133111EB & _M64
    return z ^ (z >> 31)


def _priorities(seed, draw_number, row, d):
    """31-bit priorities of a random-k draw as include/liec.h defines them."""
    G, M = 0x9E3779B97F4A7C15, 0xFFFFFFFF
    s = _mix((_mix((_mix((seed + G) & _M64) + draw_number + G) & _M64) + row + G) & _M64)
    h = torch.arange(d, dtype=torch.int64, device="cuda") ^ (s & M)
    h ^= h >> 16
    h = (h * 0x85EBCA6B) & M
    h ^= h >> 13
    h = (h + (s >> 32)) & M
    h = (h * 0xC2B2AE35) & M
    h ^= h >> 16
    return h >> 1


def _compress(v, comp, case, rng_seed, row):
    """C(v) of a vector in 64 bits."""
    if comp == "identity":
        return v.clone()
    if comp in ("sign", "blocksign"):
        off = _offsets(case) if comp == "blocksign" else [0, case["d"]]
        p = torch.empty_like(v)
        for a, b in zip(off, off[1:]):
            s = v[a:b].abs().sum() / (b - a)
            p[a:b] = torch.where(v[a:b] < 0, -s, s)
        return p
    key = v.abs() if comp == "topk" else _priorities(rng_seed, 0, row, case["d"])
    return torch.where(_top(key, case["k"]), v, torch.zeros_like(v))


def exact(case, seed):
    N = case["N"]
    wire = case["what"] == "wire"
    grads, x, e, rng_seed = _inputs(case, seed, 1 if wire else BATCHES)
    g, e = grads[0], e.double()
    if wire:
        p = torch.stack([_compress(g[i].double(), case["worker"], case, rng_seed, i) for i in range(N)])
        if case["worker"] == "sign":
            return None, p
        return None, None, p
    if case["what"] == "average":
        v, mean = torch.zeros_like(e), torch.zeros_like(e)
        for i in range(N):
            v += g[i]
            mean += x[i]
        v = v / N + e
        return (mean / N - case["lr"] * v).expand(N, -1), torch.zeros_like(e)
    v = torch.zeros_like(e)
    for i in range(N):
        v += _compress(g[i].double(), case["worker"], case, rng_seed, i)
    v = v / N + e
    p = _compress(v, case["server"], case, rng_seed, N)
    out = torch.empty((N, case["d"]), dtype=torch.float64, device="cuda")
    for i in range(N):
        gi = g[i].double()
        out[i] = x[i].double() - case["lr"] * (p + (gi - _compress(gi, case["worker"], case, rng_seed, i)))
    return out, v - p
