"""Performance cases of the streaming step: what a user of this library has it do, through its Python entry points.

A pass is one frame (or a short clip) through a stack of global-attention layers, one frame-wise attention, or one call of
the stateless quantizers / of score and select.  Sizes are those of the workloads in `inputs.CONFIGS` and of the tests'
ragged shapes.  Streams are brought to their steady cache length before they are timed, as a running stream is; a clip from
an empty cache is its own case.  The keep lists and the re-quantized cache of a step are private to the context; they are
seen through the attention outputs of the frames (and passes) that follow.
"""
import math

import torch

from paper_2602_21780_amd import xsv
from paper_2602_21780_amd.inputs import FrameSource, StreamSpec

DEV = "cuda:0"
D = 64        # channels per head: the one head dimension the library is built for
RING = 4      # distinct frames a stream cycles through once it is steady

_STREAM = dict(kind="stream", layers=1, heads=16, tokens=1374, special=5, budget=4096, bits=4, group=64, pool=16,
               score_mode=0, value_mode=0, overlap=1, calls="step", frames=1, drift=False, outliers=6, gain=8.0)


def _stream(name, **kw):
    return dict(_STREAM, name=name, **kw)


def listed():
    return [
        # Smallest: one step of the tiny configuration (2 heads, 64 tokens, budget 256).  Launches and host time.
        _stream("tiny-step", heads=2, tokens=64, budget=256, group=32, outliers=4),
        # A ragged stack of middle size: odd head count, a token count that is no multiple of anything, every head keeping
        # its own top-k, 32-token groups; driven stage by stage (attend, score_prune, quantize), as a model that puts work of
        # its own between the stages does.
        _stream("ragged-per-head-stages", layers=4, heads=5, tokens=282, special=4, budget=700, group=32, pool=1, score_mode=1,
                calls="stages"),
        # Values quantized once, 2 bits, 32-channel groups, tokens no multiple of a tile, deferred joins.
        _stream("ragged-2bit-quantize-once", layers=6, heads=12, tokens=777, budget=3000, bits=2, group=32, value_mode=1,
                overlap=2, outliers=8, gain=12.0),
        # One VGGT-shaped layer whose budget is below two frames: nothing of the middle survives (k = 0).
        _stream("one-layer-below-budget", budget=2048),
        # The 24-layer stack at 1374 tokens, budget 4096, 4 bits: one frame with deferred joins and arguments marshalled
        # once - the headline workload.
        _stream("stack-frame-deferred", layers=24, overlap=2, calls="packed", drift=True),
        # The same in the library's default sequencing, called as the README shows it: the plain way to use the library.
        _stream("stack-frame-default", layers=24, drift=True),
        # The same with all layers per launch.
        _stream("stack-frame-batched", layers=24, calls="batch", drift=True),
        # Aggressive compression of a non-square input: 1041 tokens, 2 bits, budget 8192 (long keys, most of them kept).
        _stream("stack-frame-2bit", layers=24, tokens=1041, budget=8192, bits=2, outliers=8, gain=12.0),
        # The uncompressed baseline: an unbounded bf16 cache filled from empty by a clip of 16 frames (1374 to 21984 keys).
        _stream("bf16-clip-from-empty", layers=4, budget=0, bits=16, frames=16),
        # Frame-wise attention of the alternating backbone, one layer: the frame's own tokens only.
        dict(name="frame-attention", kind="frame", heads=16, tokens=1374),
        # The stateless quantizers on keys and values of a cache's size (studies of the quantizer, other caches).
        dict(name="quantize-keys-values", kind="quantize", heads=16, tokens=4096, bits=4, group=64),
        # Score and select on bf16 keys outside a context (the allocation-free score, then the keep list).
        dict(name="score-select", kind="select", heads=16, tokens=1374, special=5, pool=16, middle=2722, keep=1348),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["stream", "frame", "quantize", "select"], [9, 1, 1, 1])[0]
    if kind == "frame":
        return dict(kind="frame", heads=rng.randint(1, 16), tokens=_log_int(rng, 33, 2000))
    if kind == "quantize":
        return dict(kind="quantize", heads=rng.randint(1, 16), tokens=_log_int(rng, 64, 8192), bits=rng.choice([2, 4]),
                    group=rng.choice([32, 64]))
    if kind == "select":
        n, middle = _log_int(rng, 64, 1374), _log_int(rng, 64, 8000)
        return dict(kind="select", heads=rng.randint(1, 16), tokens=n, special=rng.randint(0, 5), pool=rng.choice([1, 4, 16, 64]),
                    middle=middle, keep=rng.randint(1, middle - 1))
    most = max(work(c)["flops"] for c in listed())
    while True:
        c = dict(_STREAM, layers=_log_int(rng, 1, 24), heads=rng.randint(1, 16), tokens=_log_int(rng, 48, 1374),
                 special=rng.randint(0, 5), bits=rng.choice([2, 4, 4, 16]), group=rng.choice([32, 64, 64]),
                 pool=rng.choice([1, 4, 16, 16, 64]), score_mode=rng.choice([0, 0, 0, 1]), value_mode=rng.choice([0, 0, 0, 1]),
                 overlap=rng.choice([0, 1, 1, 2]), calls=rng.choice(["step", "step", "packed", "stages", "batch"]),
                 frames=1, drift=rng.random() < 0.5, outliers=rng.choice([4, 6, 8]), gain=rng.choice([8.0, 12.0]))
        if rng.random() < 0.15:    # an unbounded cache filled by a clip
            c.update(budget=0, frames=rng.randint(2, 12))
        else:                      # a budget of one and a half to eight frames
            c.update(budget=int(c["tokens"] * rng.uniform(1.5, 8.0)))
        if c["bits"] == 16:
            c.update(group=64, value_mode=0)
        if work(c)["flops"] <= most:
            return c


# ---- the length of a stream's cache (token counting of the method) ------------------------------------------------

def _next_len(c, T, frames_seen):
    n = c["tokens"]
    if c["budget"] == 0 or T + n <= c["budget"] or frames_seen == 0:
        return T + n
    middle = T - n
    return 2 * n + min(max(0, c["budget"] - 2 * n), middle)


def _steps(c):
    """Cache lengths (before, after) of the steps of one pass."""
    T, seen, steps = 0, 0, []
    warm = 0 if c["budget"] == 0 else _warm_frames(c)
    for f in range(warm + c["frames"]):
        after = _next_len(c, T, seen)
        if f >= warm:
            steps.append((T, after))
        T, seen = after, seen + 1
    return steps


def _warm_frames(c):
    """Frames until the cache has reached its steady length and has been pruned at least once more."""
    return max(2, -(-c["budget"] // c["tokens"])) + 2


def _spec(c, seed):
    return StreamSpec("case", c.get("layers", 1), c["heads"], D, c["tokens"], min(c.get("special", 0), c["tokens"]), 1000,
                      c.get("budget", 0), c.get("bits", 16), c.get("group", 64), c.get("pool", 16), seed, True,
                      c.get("outliers", 6), c.get("gain", 8.0), c.get("drift", False))


# ---- inputs, contexts, handles -----------------------------------------------------------------------------------

def prepare(case, seed):
    c = case
    src = FrameSource(_spec(c, seed), DEV)
    H, n = c["heads"], c["tokens"]
    if c["kind"] == "quantize":
        _, k, v = src.frame(0)
        return dict(case=c, k=k[0].contiguous(), v=v[0].contiguous())
    if c["kind"] == "select":
        q, _, _ = src.frame(0)
        keys = FrameSource(_spec(dict(c, tokens=c["middle"]), seed + 1), DEV).frame(0)[1][0].contiguous()
        return dict(case=c, q=q[0].contiguous(), keys=keys, scores=torch.empty(c["middle"], dtype=torch.float32, device=DEV))
    if c["kind"] == "frame":
        q, k, v = src.frame(0)
        ctx = xsv.Context(1, H, D, n, 0, 2 * n, 16, 64)
        return dict(case=c, ctx=ctx, q=q[0], k=k[0], v=v[0], out=torch.empty((H, n, D), dtype=torch.bfloat16, device=DEV))
    L = c["layers"]
    ctx = xsv.Context(L, H, D, n, min(c["special"], n), c["budget"], c["bits"], c["group"], pool_size=c["pool"],
                      max_frames=c["frames"], score_mode=c["score_mode"], value_mode=c["value_mode"])
    ctx.set_overlap(c["overlap"])
    clip = c["budget"] == 0
    n_out = c["frames"] if clip else 1
    out = torch.empty((n_out, L, H, n, D), dtype=torch.bfloat16, device=DEV)
    if not clip:
        for f in range(_warm_frames(c)):
            q, k, v = src.frame(f)
            for l in range(L):
                ctx.step(l, q[l], k[l], v[l], out[0, l])
            ctx.join()
    first = 0 if clip else _warm_frames(c)
    ring = []
    for f in range(first, first + (c["frames"] if clip else RING)):
        q, k, v = src.frame(f)
        o = out[f if clip else 0]
        if c["calls"] == "packed":
            ring.append((q, k, v, [ctx.pack_step(q[l], k[l], v[l], o[l]) for l in range(L)]))
        elif c["calls"] == "batch":
            ring.append((q, k, v, ctx.pack_layers(q, k, v, o)))
        else:
            ring.append((q, k, v, [(q[l], k[l], v[l], o[l]) for l in range(L)]))
    return dict(case=c, ctx=ctx, out=out, ring=ring, clip=clip, at=0)


def _frame(ctx, c, layers):
    if c["calls"] == "packed":
        for l, packed in enumerate(layers):
            ctx.step_packed(l, packed)
    elif c["calls"] == "batch":
        ctx.step_all_layers(packed=layers)
    elif c["calls"] == "stages":
        for l, (q, k, v, o) in enumerate(layers):
            ctx.dequant_attend(l, q, k, v, o)
            ctx.score_prune(l, q)
            ctx.quantize(l, k, v)
    else:
        for l, (q, k, v, o) in enumerate(layers):
            ctx.step(l, q, k, v, o)
    if c["overlap"] == 2:
        ctx.join()


def run(state):
    c = state["case"]
    if c["kind"] == "quantize":
        return [xsv.quantize_k(state["k"], c["bits"], c["group"]), xsv.quantize_v(state["v"], c["bits"], c["group"])]
    if c["kind"] == "select":
        xsv.score_noalloc(state["q"], state["keys"], c["special"], c["pool"], state["scores"])
        return [state["scores"], xsv.topk_keep(state["scores"], c["keep"], c["tokens"], c["tokens"])]
    ctx = state["ctx"]
    if c["kind"] == "frame":
        return ctx.frame_attend(state["q"], state["k"], state["v"], state["out"])
    if state["clip"]:
        ctx.reset()
        for frame in state["ring"]:
            _frame(ctx, c, frame[3])
    else:
        _frame(ctx, c, state["ring"][state["at"] % RING][3])
        state["at"] += 1
    return state["out"]


# ---- what a pass cannot do without ---------------------------------------------------------------------------------

def work(case):
    c = case
    H, n = c["heads"], c["tokens"]
    if c["kind"] == "frame":
        return {"bytes": 4 * 2 * n * H * D, "flops": 4 * n * n * H * D}
    if c["kind"] == "quantize":      # bf16 in, a byte per code and two fp32 per group out, keys and values
        T, G = n, c["group"]
        return {"bytes": 2 * H * T * D * 3 + 8 * H * (-(-T // G) * D + T * (D // G)), "flops": 2 * 4 * H * T * D}
    if c["kind"] == "select":
        P = c["middle"]
        return {"bytes": 2 * H * D * (n + P) + 4 * P + 4 * (2 * n + c["keep"]), "flops": 2 * H * D * (n + P) // 2}
    row = 2.0 if c["bits"] == 16 else c["bits"] / 8.0 + 8.0 / c["group"]    # bytes per cached element
    nbytes, flops = 0.0, 0.0
    for T, after in _steps(c):
        written = after if c["budget"] else n        # an unbounded cache only appends
        nbytes += c["layers"] * H * D * (4 * 2 * n + 2 * row * (T + written))
        flops += c["layers"] * H * D * 4.0 * n * (T + n)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "quantize":
        return "exact"               # codes, scales and zero points are defined bit for bit
    if case["kind"] == "select":
        return {"rel": 8e-7}         # fp32 sums: 1.8e-7 from the same sums in fp64; the keep list is whole numbers
    # bf16 probabilities and outputs, partial sums in fp16: the same streams with their keys cut into other ranges differ by
    # up to 2.4e-3 (largest single value 0.037 of the rms), frame-wise attention from fp64 by 2.0e-3
    return {"rel": 9e-3, "max": 0.15}
