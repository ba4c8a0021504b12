"""The workloads whose speed matters, as data: one case is one network with its options, one pass is one optimizer
step of it (`PipeMare.step`, called once per microbatch) on batches that are resident on the GPU.

The range is what the engine takes: chains of Linear units, fine-grained causal Transformers and ResNet-shaped
networks; bf16 and fp32; momentum SGD and AdamW; one or several microbatches per step, clipping, recomputation,
stochastic delays; captured graphs and eager launches.  `listed()` holds the benchmark configurations and, between
them, small, ragged and optional ones; `draw()` gives more of the same ranges.

A pass returns the state arrays of the recurrence as they lie in the caller's arena (master weights, gradients,
moments, delta accumulator, corrected backward weights): views, no copies.
"""
import collections
import math

import numpy as np
import torch

import paper_1910_05124_amd as pm

Unit = collections.namedtuple("Unit", "kind n_in n_out act stage")

_streams = {}


def _stream():
    """The program's one training stream (a captured step needs a stream of its own)."""
    dev = torch.cuda.current_device()
    if dev not in _streams:
        _streams[dev] = torch.cuda.Stream()
    return _streams[dev]


# ------------------------------------------------------------------------------------------------------ cases
def _chain(name, dtype, widths_in, width, depth, n_out, rows, act, loss, **kw):
    return dict(name=name, family="chain", dtype=dtype, n_in=widths_in, width=width, depth=depth, n_out=n_out, rows=rows,
                act=act, loss=loss, **kw)


def _tfm(name, dtype, layers, d, heads, ff, vocab, seq, batch, **kw):
    return dict(name=name, family="transformer", dtype=dtype, layers=layers, d=d, heads=heads, ff=ff, vocab=vocab, seq=seq,
                batch=batch, **kw)


def _cnn(name, dtype, blocks, image, classes, batch, **kw):
    return dict(name=name, family="resnet", dtype=dtype, blocks=blocks, image=image, classes=classes, batch=batch, **kw)


def listed():
    return [
        # the smallest call: the 4-stage fp32 regression net (64 wide, 16 rows), all launches and latency
        _chain("mlp4_f32", "f32", 64, 64, 3, 1, 16, "relu", "mse", graph=True),
        # an fp32 classifier of ordinary size with an odd row count
        _chain("mlp8x512_f32", "f32", 784, 512, 8, 10, 100, "gelu", "xent", graph=True),
        # the 16-stage bf16 MLP of the benchmark: a long chain of small products, then 0.5 GB of update
        _chain("mlp16_bf16", "bf16", 1024, 1024, 16, 10, 128, "gelu", "xent", graph=True),
        # a wide bf16 MLP fed with a ragged thousand of rows, launched eagerly
        _chain("mlp6x2048_bf16", "bf16", 1000, 2048, 6, 1000, 1000, "relu", "xent", graph=False),
        # a small fp32 Transformer with 32-wide heads, as used to check a recipe before the bf16 run
        _tfm("tfm2x256_f32", "f32", 2, 256, 8, 1024, 2000, 64, 8, opt="adamw", graph=True),
        # translation-sized bf16 batch with nothing round about it: 100 tokens, odd vocabulary, 5 heads
        _tfm("tfm4x320_ragged", "bf16", 4, 320, 5, 1280, 10007, 100, 24, opt="adamw", graph=True),
        # the 6-layer Transformer of the benchmark
        _tfm("tfm6x512_bf16", "bf16", 6, 512, 8, 2048, 8192, 128, 32, opt="adamw", graph=True),
        # the same network with recomputation in segments of 6 stages
        _tfm("tfm6x512_recompute", "bf16", 6, 512, 8, 2048, 8192, 128, 32, opt="adamw", segment=6, graph=True),
        # four microbatches per step with clipping of the global gradient norm
        _tfm("tfm3x768_micro4", "bf16", 3, 768, 12, 3072, 16000, 256, 8, opt="adamw", micro=4, clip=25.0, graph=False),
        # the largest: the 12-layer Transformer of the benchmark, every unit a stage of its own
        _tfm("tfm12x1024_bf16", "bf16", 12, 1024, 16, 4096, 32000, 512, 16, opt="adamw", ln_stage=True, graph=True),
        # the ResNet-20 shape of the benchmark
        _cnn("resnet20_bf16", "bf16", 3, 32, 10, 128, graph=True),
        # a shallower one on 28 x 28 images and a last, incomplete batch
        _cnn("resnet14_ragged", "bf16", 2, 28, 10, 37, graph=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        c = _draw_one(rng)
        w, top = work(c), work(listed()[9])
        # fp32 products run on the vector units and attention outside the matrix path on one thread per row: an order
        # of magnitude dearer each, so they are drawn an order of magnitude and more smaller
        f32 = c["dtype"] == "f32"
        if w["flops"] * (40 if f32 else 2) <= top["flops"] and w["bytes"] * 2 <= top["bytes"] and _ring_bytes(c) < 12e9:
            return c


def _draw_one(rng):
    family = rng.choice(["chain", "chain", "chain", "transformer", "transformer", "transformer", "resnet", "resnet"])
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    common = dict(opt=rng.choice(["sgdm", "adamw"]), graph=rng.random() < 0.75)
    if rng.random() < 0.15:
        common.update(micro=rng.randint(2, 4), graph=False)
    if rng.random() < 0.15:
        common["clip"] = 25.0
    pick = rng.random()
    if pick < 0.1:
        common["segment"] = rng.randint(2, 6)
    elif pick < 0.2:
        common["tau_max"] = rng.randint(1, 40)
    if family == "chain":
        # bf16 matrices have rows of whole 16-byte pieces in earnest; fp32 ones anything
        step = 8 if dtype == "bf16" else 1
        c = _chain("", dtype, _log(rng, 16, 2048) // step * step, _log(rng, 32, 2048 if dtype == "bf16" else 768) // step * step,
                   rng.randint(2, 16), rng.choice([1, 10, 100, 1000]), _log(rng, 4, 4096 if dtype == "bf16" else 512),
                   rng.choice(["relu", "gelu"]), "xent", **common)
        if c["n_out"] == 1:
            c["loss"] = "mse"
    elif family == "transformer":
        dh = rng.choice([64, 64, 64, 32])
        heads = rng.randint(1, 16 if dtype == "bf16" else 6)
        d = dh * heads
        if dtype == "bf16" and dh == 64 and rng.random() < 0.6:
            seq = 32 * rng.randint(1, 16)
        else:
            seq = _log(rng, 8, 8192 // (dh + 1))
        tokens = _log(rng, 128, 8192 if dtype == "bf16" else 1024)
        c = _tfm("", dtype, rng.randint(1, 6), d, heads, d * rng.choice([2, 4]), _log(rng, 200, 32000), seq,
                 max(1, tokens // seq), **common)
    else:
        c = _cnn("", dtype, rng.randint(1, 3), 4 * rng.randint(4, 12), rng.choice([10, 100]),
                 _log(rng, 4, 256 if dtype == "bf16" else 16), **common)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------------ networks
def _units(c):
    """(units, stages) of a case: one stage per weight matrix or convolution."""
    if c["family"] == "chain":
        w = [c["n_in"]] + [c["width"]] * c["depth"]
        u = [Unit("linear", w[j], w[j + 1], c["act"], j + 1) for j in range(c["depth"])]
        # the head is a stage of its own in the regression net and rides in the last stage of a classifier
        last = c["depth"] + 1 if c["loss"] == "mse" else c["depth"]
        return u + [Unit("linear", c["width"], c["n_out"], "none", last)], last
    if c["family"] == "transformer":
        d, own = c["d"], bool(c.get("ln_stage"))
        u, st = [Unit("embed", c["vocab"], d, "none", 1)], 1

        def add(kind, n_in, n_out, act, new):
            nonlocal st
            st += new
            u.append(Unit(kind, n_in, n_out, act, st))

        for _ in range(c["layers"]):
            add("layernorm", d, d, "none", True)
            add("linear", d, d, "none", own)
            for _ in range(3):
                add("linear", d, d, "none", True)
            add("layernorm", d, d, "none", True)
            add("linear", d, c["ff"], "relu", own)
            add("linear", c["ff"], d, "none", True)
        add("layernorm", d, d, "none", True)
        add("linear", d, c["vocab"], "none", own)
        return u, st
    u, ch = [Unit("conv3x3", 3, 16, "relu", 1)], 16
    for group in range(3):
        for block in range(c["blocks"]):
            cin = ch
            if group > 0 and block == 0:
                ch *= 2
            u.append(Unit("conv3x3", cin, ch, "relu", len(u) + 1))
            u.append(Unit("conv3x3", ch, ch, "relu", len(u) + 1))
    u.append(Unit("linear", 64, c["classes"], "none", len(u) + 1))
    return u, len(u)


def _parts(u):
    """Values of a unit's first part (matrix, table, gain, kernel) and of its second."""
    if u.kind == "embed":
        return u.n_in * u.n_out, 0
    if u.kind == "layernorm":
        return u.n_out, u.n_out
    if u.kind == "conv3x3":
        return u.n_out * 9 * u.n_in, 2 * u.n_out
    return u.n_out * u.n_in, u.n_out


def _delays(c, stages):
    tau_f, tau_b = pm.pm_delays(stages, c.get("micro", 1), "pipemare")
    tau_r = pm.pm_recompute_delays(stages, c["segment"], c.get("micro", 1), tau_b) if c.get("segment") else None
    return tau_f, tau_b, tau_r


def _ring_bytes(c):
    units, stages = _units(c)
    tau_f, _, _ = _delays(c, stages)
    esz = 2 if c["dtype"] == "bf16" else 4
    return sum(sum(_parts(u)) * ((c["tau_max"] if "tau_max" in c else tau_f[u.stage - 1]) + 1) * esz for u in units)


def _flat(units):
    """Padded length of the engine's flat arrays: a unit's second part starts at a multiple of 8 values, a unit at a
    multiple of 2048."""
    return sum(((nw + 7) // 8 * 8 + nb + 2047) // 2048 * 2048 for nw, nb in map(_parts, units))


def _init(units, gen):
    """Initial weights as a user's program draws them: uniform within 1 / sqrt(fan_in) (He's bound in front of an
    activation), a normal embedding, LayerNorm and folded normalisation near their usual starting points."""
    def uniform(n, bound):
        return (torch.rand(n, device="cuda", generator=gen) * 2 - 1) * bound

    out = []
    for u in units:
        nw, nb = _parts(u)
        if u.kind == "embed":
            v = torch.randn(nw, device="cuda", generator=gen) / math.sqrt(u.n_out)
        elif u.kind == "layernorm":
            v = uniform(nw + nb, 0.1)
            v[:nw] += 1.0
        elif u.kind == "conv3x3":
            v = torch.cat([uniform(nw, math.sqrt(6.0 / (9 * u.n_in))), 0.5 + uniform(u.n_out, 0.05), uniform(u.n_out, 0.1)])
        else:
            bound = math.sqrt(6.0 / u.n_in) if u.act in ("relu", "gelu") else math.sqrt(1.0 / u.n_in)
            v = torch.cat([uniform(nw, bound), uniform(nb, math.sqrt(1.0 / u.n_in))])
        out.append(v.cpu().numpy())
    return out


def _batch(c, gen):
    if c["family"] == "chain":
        x = torch.randn(c["rows"], c["n_in"], device="cuda", generator=gen)
        if c["loss"] == "mse":
            return x, torch.randn(c["rows"], c["n_out"], device="cuda", generator=gen)
        return x, torch.randint(c["n_out"], (c["rows"],), device="cuda", generator=gen, dtype=torch.int32)
    if c["family"] == "transformer":
        # token ids with the rank-frequency law of natural text, target = next token
        p = torch.arange(1, c["vocab"] + 1, device="cuda", dtype=torch.float64) ** -1.1
        cdf = torch.cumsum(p / p.sum(), 0)
        r = torch.rand(c["batch"], c["seq"] + 1, device="cuda", generator=gen, dtype=torch.float64)
        ids = torch.searchsorted(cdf, r).clamp_(max=c["vocab"] - 1).to(torch.int32)
        return ids[:, :-1].contiguous(), ids[:, 1:].contiguous()
    x = torch.randn(c["batch"], 3, c["image"], c["image"], device="cuda", generator=gen)
    return x, torch.randint(c["classes"], (c["batch"],), device="cuda", generator=gen, dtype=torch.int32)


# ------------------------------------------------------------------------------------------------------ one pass
def prepare(case, seed):
    """The engine of the case, two optimizer steps into its run (the rings, the delta accumulator and, where the step
    is a captured graph, the graph are those of a run under way), and its batches."""
    c = case
    units, stages = _units(c)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    tau_f, tau_b, tau_r = _delays(c, stages)
    micro = c.get("micro", 1)
    # small constant base step: the run may go on for thousands of passes over the same few batches
    sched = pm.make_sched(kind="const", base=1e-4, K=40000)
    stochastic = dict(tau_max=c["tau_max"], seed=seed) if "tau_max" in c else None
    opts = pm.make_opts(opt=c.get("opt", "sgdm"), beta1=0.9, beta2=0.98, D=0.5, N=micro, dtype=c["dtype"],
                        loss=c.get("loss", "xent"), clip_norm=c.get("clip", 0.0), microbatch=c.get("rows") or c["batch"],
                        use_graph=bool(c["graph"]), arch=c["family"], n_heads=c.get("heads", 0), seq_len=c.get("seq", 0),
                        image_size=c.get("image", 0), tau_recomp=tau_r, segment_size=c.get("segment", 0),
                        stochastic=stochastic)
    weights = _init(units, gen)
    batches = [_batch(c, gen) for _ in range(micro)]
    torch.cuda.current_stream().synchronize()
    stream = _stream()
    with torch.cuda.stream(stream):
        engine = pm.PipeMare(units, stages, tau_f, tau_b, sched, opts, weights, stream=stream)
    n = _flat(units)
    start = -engine.arena.data_ptr() % 256
    names = ["weights", "grads", "moment1"] + (["moment2"] if c.get("opt") == "adamw" else []) + ["delta"]
    arrays = {k: engine.arena[start + 4 * n * i:start + 4 * n * (i + 1)].view(torch.float32) for i, k in enumerate(names)}
    at, esz = start + 4 * n * len(names), 2 if c["dtype"] == "bf16" else 4
    arrays["corrected"] = engine.arena[at:at + esz * n].view(torch.bfloat16 if esz == 2 else torch.float32)
    if c.get("opt") == "adamw":
        # the sign of an Adam step whose gradient is rounding noise is noise itself: the accumulator of such steps says
        # nothing (two orders of summation differ by 1.5 % there), the corrected weights made from it do
        del arrays["delta"]
    state = {"engine": engine, "batches": batches, "out": arrays}
    for _ in range(2):
        run(state)
    return state


def run(state):
    for x, y in state["batches"]:
        state["engine"].step(x, y)
    return state["out"]


# ------------------------------------------------------------------------------------------------------ what a pass needs
def work(case):
    """Bytes: the state arrays read and written once, the gradient written, the delayed forward and backward weights
    read, the new version and the corrected weights written, the batch read.  Operations: every product's forward,
    weight gradient and (but for the first unit) data gradient, the rebuilt forward of recomputation, the causal
    attention core."""
    c = case
    units, _ = _units(c)
    micro, adam, esz = c.get("micro", 1), c.get("opt") == "adamw", 2 if c["dtype"] == "bf16" else 4
    n = sum(sum(_parts(u)) for u in units)
    byts = n * (8.0 * (4 if adam else 3) + 4 + 4 * esz)
    flops = 0.0
    again = 1 if c.get("segment") else 0
    if c["family"] == "chain":
        for i, u in enumerate(units):
            flops += (2 + (i > 0) + again) * 2.0 * c["rows"] * u.n_in * u.n_out
        byts += micro * 4.0 * c["rows"] * (c["n_in"] + 1)
    elif c["family"] == "transformer":
        tok = c["batch"] * c["seq"]
        flops += (3 + again) * 2.0 * tok * sum(u.n_in * u.n_out for u in units if u.kind == "linear")
        flops += (6 + 2 * again) * c["layers"] * float(c["batch"]) * c["d"] * c["seq"] ** 2
        byts += micro * 8.0 * tok
    else:
        side = c["image"]
        for i, u in enumerate(units[:-1]):
            if i and u.n_out == 2 * u.n_in:
                side //= 2
            flops += (2 + (i > 0) + again) * 2.0 * c["batch"] * side * side * 9 * u.n_in * u.n_out
        flops += 6.0 * c["batch"] * 64 * c["classes"]
        byts += micro * 4.0 * c["batch"] * 3 * c["image"] ** 2
    return {"bytes": byts, "flops": micro * flops}


def tolerance(case):
    """Measured with the hidden units, heads and channels of a network permuted, i.e. every contraction summed in another
    order: the gradients then differ by at most 2.6e-6 (fp32), 2.5e-3 (bf16 Transformers and residual networks) and
    1.0e-2 (bf16 chains, which have no residual stream to keep a rounding from passing through every unit); four times
    that."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 4e-2 if case["family"] == "chain" else 1e-2}
