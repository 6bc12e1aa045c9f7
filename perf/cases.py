"""The work a user of this library has it do, as measurable cases.

A case is one call sequence through the public entry points of the binding: a pipeline-stage step (forward and
backward of `layers` decoder layers over `micro` micro-batches), one direction of one layer, or the forward pass that
allocates nothing.  Shapes are the decoder layers of the repository's workloads, benchmark and tests and generic
smaller ones; values are what training meets: activations and gradients of unit variance, projections initialised
with variance 2 / (5 hidden), norm gains near one.

Fields: op  step       hh_stage_step, gradients summed over the micro-batches
            1f1b       hh_stage_step_1f1b with `live` micro-batches alive
            fwd        hh_layer_fwd that saves for a backward pass
            infer      hh_layer_fwd without a saved block (forward only)
            noalloc    hh_layer_fwd_noalloc
            bwd        hh_layer_bwd on what a forward call has saved
        dtype          "bf16" (activations and weights bf16, gradients fp32) or "f32"
        hidden, heads, kv_heads, head_dim, ffn, seq, batch, layers, micro, live
        packed         wq|wk|wv and w_gate|w_up (and their gradients) in one allocation each
        accumulate     gradients are added to what the buffers hold, instead of written
"""
from __future__ import annotations

import math

import torch

from paper_2405_16256_amd import binding as hh

DEVICE = "cuda:0"
ORDER = ("name", "op", "dtype", "hidden", "heads", "kv_heads", "head_dim", "ffn", "seq", "batch", "layers", "micro", "live",
         "packed", "accumulate")


def _case(name, op, dtype, hidden, heads, kv_heads, head_dim, ffn, seq, batch=1, layers=1, micro=1, live=0, packed=True,
          accumulate=False):
    return dict(zip(ORDER, (name, op, dtype, hidden, heads, kv_heads, head_dim, ffn, seq, batch, layers, micro, live or micro,
                            packed, accumulate)))


def listed():
    return [
        # The smallest configuration of the repository, fp32: a correctness run on a laptop-sized model.  A handful of
        # microseconds of arithmetic, so launches and latency count.
        _case("f32 tiny layer step", "step", "f32", 256, 4, 4, 64, 688, 128),
        # fp32 at a size where arithmetic counts: the reference-precision run a user compares a bf16 run with.
        _case("f32 hidden-1024 step", "step", "f32", 1024, 8, 2, 128, 2048, 700),
        # The tiny model's stage in bf16, four layers and eight micro-batches in one-forward-one-backward order: what a
        # functional test of a pipeline runs.
        _case("tiny 4-layer 1f1b stage", "1f1b", "bf16", 256, 4, 4, 64, 704, 128, layers=4, micro=8, live=2),
        # Forward of a small layer in a serving loop that may not allocate; grouped queries, odd length.
        _case("small no-alloc forward", "noalloc", "bf16", 1024, 8, 2, 128, 2048, 700),
        # A small research model: head_dim 64, grouped queries, ragged length, separately allocated projections, two
        # samples, gradients summed over three micro-batches.
        _case("small ragged 2-layer step", "step", "bf16", 512, 8, 2, 64, 768, 1100, batch=2, layers=2, micro=3, packed=False),
        # A short prompt through a 7B-class layer, forward only: prefill.
        _case("7B-class prefill of 333", "infer", "bf16", 4096, 32, 32, 128, 11008, 333),
        # A tensor-parallel share with a ragged token count.
        _case("hidden-4096 share of 3300", "step", "bf16", 4096, 8, 8, 128, 4096, 3300),
        # 7B-class layer, forward and backward in training (gradients accumulate over calls).
        _case("7B-class layer step", "step", "bf16", 4096, 32, 32, 128, 11008, 2048, accumulate=True),
        # Backward alone of a hidden-8192 layer at an eighth tensor-parallel share: 8 query heads on one key/value head.
        _case("hidden-8192 GQA share bwd", "bwd", "bf16", 8192, 8, 1, 128, 3584, 4096, accumulate=True),
        # The benchmark's layer: 140B-class at an eighth tensor-parallel share.
        _case("140B-class share step", "step", "bf16", 12288, 12, 12, 128, 4096, 4096, accumulate=True),
        # The whole hidden-8192 layer, no tensor parallelism.
        _case("hidden-8192 GQA layer step", "step", "bf16", 8192, 64, 8, 128, 28672, 4096),
        # A pipeline stage in earnest: four layers of the benchmark's shape, eight micro-batches, two of them alive.
        _case("140B-class stage 1f1b", "1f1b", "bf16", 12288, 12, 12, 128, 4096, 4096, layers=4, micro=8, live=2),
    ]


def _flops(c):
    """Model flops of one forward pass of one layer on one micro-batch; a backward pass is twice that."""
    a, akv, t = c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"], c["seq"] * c["batch"]
    gemm = t * (2.0 * (2 * a + 2 * akv) * c["hidden"] + 6.0 * c["hidden"] * c["ffn"])
    return gemm + 4.0 * c["head_dim"] * c["batch"] * c["heads"] * (c["seq"] * (c["seq"] + 1) / 2)


def _passes(c):
    """(forward passes, backward passes) of a layer in one run."""
    n = c["layers"] * c["micro"]
    return (n if c["op"] != "bwd" else 0, n if c["op"] in ("step", "1f1b", "bwd") else 0)


def _total_flops(c):
    f, b = _passes(c)
    return (f + 2 * b) * _flops(c)


def _params(c):
    a, akv = c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"]
    return 2 * c["hidden"] + (2 * a + 2 * akv) * c["hidden"] + 3 * c["ffn"] * c["hidden"]


def _state_bytes(c):
    """A generous bound of what a state holds on the GPU."""
    es = 2 if c["dtype"] == "bf16" else 4
    a, akv, t = c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"], c["seq"] * c["batch"]
    saved = t * (4 * c["hidden"] + 2 * a + 2 * akv + 2 * c["ffn"]) * es
    return c["layers"] * _params(c) * (es + 4) + (c["live"] * c["layers"] + 3) * saved + 4 * c["micro"] * t * c["hidden"] * es


def draw(rng):
    def log(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    def multiple(of, lo, hi):
        return min(hi, max(of, int(round(log(lo, hi) / of)) * of))

    most = {"bf16": max(_total_flops(c) for c in listed() if c["dtype"] == "bf16"),
            "f32": max(_total_flops(c) for c in listed() if c["dtype"] == "f32")}
    while True:
        dtype = "f32" if rng.random() < 0.15 else "bf16"
        op = rng.choice(("step", "step", "step", "1f1b", "fwd", "infer", "bwd", "noalloc"))
        d = rng.choice((64, 128, 128))
        of = 64 if dtype == "bf16" else 8
        top_h, top_f, top_s = (12288, 28672, 4096) if dtype == "bf16" else (1024, 2048, 1024)
        if op == "noalloc":                     # has to fit the library's own scratch array
            top_h, top_f, top_s = 1024, 2048, 700
        hidden = multiple(of, 128, top_h)
        heads = max(1, min(64, int(round(hidden / d * rng.choice((0.125, 0.25, 0.5, 1.0, 1.0))))))
        if op == "noalloc":
            heads = min(heads, 1024 // d)
        kv_heads = heads
        if rng.random() < 0.4:
            kv_heads = rng.choice([k for k in range(1, heads + 1) if heads % k == 0])
        ffn = multiple(of, max(of, hidden // 3), max(of, min(top_f, int(hidden * 3.5))))
        seq = int(round(log(17, top_s)))
        batch = rng.choice((1, 1, 1, 2, 4)) if op != "noalloc" else 1
        layers, micro, live = 1, 1, 1
        if op in ("step", "1f1b"):
            layers, micro = rng.choice((1, 1, 2, 3, 4)), rng.choice((1, 1, 2, 4, 8))
            live = micro if op == "step" else rng.randint(1, micro)
        c = _case("", op, dtype, hidden, heads, kv_heads, d, ffn, seq, batch, layers, micro, live, packed=rng.random() < 0.75,
                  accumulate=op in ("step", "1f1b", "bwd") and rng.random() < 0.5)
        del c["name"]
        if _total_flops(c) <= most[dtype] and _state_bytes(c) <= 60e9:
            return c


class _Context:
    """The library's handle, freed with its owner."""

    def __init__(self):
        self.ptr = hh.hh_ctx_create(0)

    def __del__(self):
        hh.hh_ctx_destroy(self.ptr)


def _cfg(c):
    return hh.make_cfg(c["hidden"], c["heads"], c["head_dim"], c["ffn"], c["seq"], c["batch"],
                       dtype=hh.HH_BF16 if c["dtype"] == "bf16" else hh.HH_F32, n_kv_heads=c["kv_heads"])


def prepare(case, seed):
    c = case
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)

    def normal(*shape, scale=1.0, mean=0.0):
        return torch.empty(*shape, dtype=torch.float32, device=DEVICE).normal_(mean, scale, generator=gen).to(dt)

    h, f = c["hidden"], c["ffn"]
    a, akv = c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"]
    std = math.sqrt(2.0 / (5.0 * h))
    backward = c["op"] in ("step", "1f1b", "bwd")

    def layer():
        w = {"g_attn": normal(h, scale=0.02, mean=1.0), "g_mlp": normal(h, scale=0.02, mean=1.0), "wo": normal(h, a, scale=std),
             "w_down": normal(h, f, scale=std)}
        parts = [(("wq", a), ("wk", akv), ("wv", akv)), (("w_gate", f), ("w_up", f))]
        for group in parts:
            rows = sum(n for _, n in group)
            block = normal(rows, h, scale=std) if c["packed"] else None
            at = 0
            for name, n in group:
                w[name] = block[at:at + n] if c["packed"] else normal(n, h, scale=std)
                at += n
        g = {}
        if backward:
            g = {n: torch.zeros(w[n].shape, dtype=torch.float32, device=DEVICE) for n in ("g_attn", "g_mlp", "wo", "w_down")}
            for group in parts:
                block = torch.zeros(sum(n for _, n in group), h, dtype=torch.float32, device=DEVICE) if c["packed"] else None
                at = 0
                for name, n in group:
                    g[name] = block[at:at + n] if c["packed"] else torch.zeros(n, h, dtype=torch.float32, device=DEVICE)
                    at += n
        return w, g

    s = {"case": c, "cfg": _cfg(c), "ctx": _Context()}
    hh.hh_ctx_reserve(s["ctx"].ptr, s["cfg"])
    made = [layer() for _ in range(c["layers"])]
    s["w"], s["g"] = [w for w, _ in made], [g for _, g in made]
    s["wstruct"] = [hh.make_weights(w) for w in s["w"]]
    s["gstruct"] = [hh.make_grads(g) for g in s["g"]] if backward else []
    shape = (c["batch"], c["seq"], h)
    s["x"] = [normal(*shape) for _ in range(c["micro"])]
    s["y"] = [torch.empty_like(x) for x in s["x"]]
    if backward:
        s["dy"] = [normal(*shape) for _ in range(c["micro"])]
        s["dx"] = [torch.empty_like(x) for x in s["x"]]
    if c["op"] in ("step", "1f1b"):
        pool, ws = hh.hh_stage_sizes(s["cfg"], c["layers"], c["live"])
    else:
        saved, ws = hh.hh_layer_sizes(s["cfg"])
        pool = saved if c["op"] in ("fwd", "bwd") else 0
        ws += saved if c["op"] == "infer" else 0
    if c["op"] != "noalloc":
        s["saved"] = torch.empty(pool, dtype=torch.uint8, device=DEVICE) if pool else None
        s["ws"] = torch.empty(ws, dtype=torch.uint8, device=DEVICE)
    if c["op"] == "bwd":
        hh.hh_layer_fwd(s["ctx"].ptr, s["cfg"], s["wstruct"][0], s["x"][0], s["y"][0], s["saved"], s["ws"],
                        torch.cuda.current_stream().cuda_stream)
    return s


def run(state):
    s = state
    c, cfg, ctx = s["case"], s["cfg"], s["ctx"].ptr
    stream = torch.cuda.current_stream().cuda_stream
    zero_first = not c["accumulate"]
    if c["op"] == "step":
        hh.hh_stage_step(ctx, cfg, s["wstruct"], s["x"], s["y"], s["dy"], s["dx"], s["gstruct"], zero_first, s["saved"], s["ws"], stream)
    elif c["op"] == "1f1b":
        hh.hh_stage_step_1f1b(ctx, cfg, s["wstruct"], c["live"], s["x"], s["y"], s["dy"], s["dx"], s["gstruct"], zero_first, s["saved"],
                              s["ws"], stream)
    elif c["op"] == "bwd":
        hh.hh_layer_bwd(ctx, cfg, s["wstruct"][0], s["x"][0], s["saved"], s["dy"][0], s["dx"][0], s["gstruct"][0], c["accumulate"], s["ws"],
                        stream)
        return {"dx": s["dx"], "grads": s["g"]}
    elif c["op"] == "noalloc":
        hh.hh_layer_fwd_noalloc(ctx, cfg, s["wstruct"][0], s["x"][0], s["y"][0], stream)
        return {"y": s["y"]}
    else:
        hh.hh_layer_fwd(ctx, cfg, s["wstruct"][0], s["x"][0], s["y"][0], s["saved"], s["ws"], stream)
        return {"y": s["y"]}
    return {"y": s["y"], "dx": s["dx"], "grads": s["g"]}


def work(case):
    c = case
    es = 2 if c["dtype"] == "bf16" else 4
    f, b = _passes(c)
    act = c["micro"] * c["seq"] * c["batch"] * c["hidden"] * es
    total = c["layers"] * _params(c) * es + (2 * act if f else 0)
    if b:
        total += 2 * act + c["layers"] * _params(c) * 4 * (2 if c["accumulate"] else 1)
    if c["op"] == "bwd":
        a, akv, t = c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"], c["seq"] * c["batch"]
        total += act + t * (3 * c["hidden"] + 2 * a + 2 * akv + 2 * c["ffn"]) * es
    return {"bytes": float(total), "flops": float(_total_flops(c))}


def tolerance(case):
    # Largest relative error over all outputs against the same equations in 64-bit torch autograd: fp32 path 1.6e-6;
    # bf16 path (activations and intermediate gradients rounded to bf16, fp32 sums) 5.6e-3 for one layer, 7.0e-3 for
    # two and 9.9e-3 for four, where roundings add up along the depth.
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 0.02}
