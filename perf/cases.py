"""Performance cases of the routed FFN layer: what a user's program has it do, through its public entry points.

A case is a dict of plain values.  `kind` says which path it takes:
  moe       token-choice MoE training step: route, forward, load export, backward, gate backward
  capacity  the same with the routing variants: selection bias, softmax over all experts, expert capacity
  top1      one slot per token, with the combine and the scatter folded into the last products' stores
  mod       Mixture-of-Depths training step (one expert, per-sequence capacity, residual)
  exit      a stack of early-exit layers, forward and backward (one expert each, residual)
  forward   forward only, rows gathered inside the first product: prefill and decode
Inputs have the distributions of the benchmark's workloads (workloads.py), drawn on the GPU: logits N(0,1) with
a Zipf bias over the experts, scores and activations N(0,1), weights N(0, 0.02^2), exit layers geometric.
"""
import math

import numpy as np
import torch

from paper_2505_14864_amd import binding as B
from paper_2505_14864_amd.layer import RoutedFFNLayer


def listed():
    return [
        # The smallest training step (the fp32 workload of the benchmark): every launch and host call counts.
        dict(name="moe_f32_tiny", kind="moe", dtype="f32", T=256, H=128, F=256, E=4, k=2, zipf=0.5),
        # An fp32 layer of ordinary, ragged size: debugging and reference runs of a model in full precision.
        dict(name="moe_f32_ragged", kind="moe", dtype="f32", T=1500, H=516, F=1030, E=8, k=2, zipf=1.1),
        # A small bf16 layer with sizes off every tile boundary.
        dict(name="moe_small_ragged", kind="moe", dtype="bf16", T=600, H=520, F=1032, E=8, k=2, zipf=1.1),
        # Mixtral-8x7B-shaped layer, two sequences of 2048: the headline workload and the largest case.
        dict(name="moe_mixtral", kind="moe", dtype="bf16", T=4096, H=4096, F=14336, E=8, k=2, zipf=1.1),
        # LLaMA-MoE-3.5B-shaped layer: small experts, an F that fits no tile, strongly skewed segments.
        dict(name="moe_llama", kind="moe", dtype="bf16", T=8192, H=4096, F=688, E=16, k=4, zipf=1.3),
        # Many small experts and many slots per token (the limits of the boundary): about 256 rows per expert.
        dict(name="moe_many_experts", kind="moe", dtype="bf16", T=2048, H=2048, F=1024, E=64, k=8, zipf=1.1),
        # The routing variants on an odd token count: biased selection, all-expert softmax, tokens dropped at capacity.
        dict(name="moe_capacity", kind="capacity", dtype="bf16", T=3000, H=2048, F=4096, E=16, k=2, zipf=1.1, factor=1.25),
        # Top-1 routing with the folded forward and backward.
        dict(name="moe_top1_folded", kind="top1", dtype="bf16", T=8192, H=2048, F=4096, E=8, k=1, zipf=1.1),
        # Mixture-of-Depths block: 256 of 2048 tokens per sequence, so few rows that tiles are scarce.
        dict(name="mod_block", kind="mod", dtype="bf16", T=8192, H=2048, F=8192, B=4, S=2048, cap=256),
        # Four early-exit layers, 8 x 2048 tokens, 30 % leaving per layer: dense-like products that shrink.
        dict(name="exit_stack", kind="exit", dtype="bf16", T=16384, H=2048, F=8192, layers=4, p=0.3),
        # Prefill of a Mixtral-shaped layer, an odd prompt length.
        dict(name="prefill_mixtral", kind="forward", dtype="bf16", T=1000, H=4096, F=14336, E=8, k=2, zipf=1.1),
        # One decode step of 32 sequences through the same layer: bound by reading the weights once.
        dict(name="decode_mixtral", kind="forward", dtype="bf16", T=32, H=4096, F=14336, E=8, k=2, zipf=1.1),
    ]


MAX_FLOPS = {"bf16": 4.0e12, "f32": 3.0e10}  # a drawn case stays below the largest listed one
MAX_WEIGHTS = 4.6e8                          # elements of one weight tensor, over experts and layers


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, odd_step):
    """A feature size: half the time a multiple of 128, as models have them, else any multiple of odd_step."""
    v = _log(rng, lo, hi)
    step = 128 if v >= 128 and rng.random() < 0.5 else odd_step
    return min(hi, max(step, v // step * step))


def draw(rng):
    while True:
        kind = rng.choice(["moe", "moe", "moe", "forward", "forward", "capacity", "top1", "mod", "exit"])
        dtype = "f32" if kind in ("moe", "forward") and rng.random() < 0.3 else "bf16"
        c = dict(kind=kind, dtype=dtype)
        if dtype == "f32":
            c.update(T=_log(rng, 16, 2048), H=_size(rng, 32, 1024, 4), F=_size(rng, 32, 2048, 2))
        else:
            c.update(T=_log(rng, 64, 16384), H=_size(rng, 128, 4096, 8), F=_size(rng, 128, 14336, 8))
        if kind in ("moe", "forward", "capacity", "top1"):
            E = _log(rng, 2, 16 if dtype == "f32" else 64)
            c.update(E=E, k=1 if kind == "top1" else rng.randint(1, min(E, 8)), zipf=round(rng.uniform(0.0, 2.0), 2))
        if kind == "forward":
            c["T"] = _log(rng, 1, 2048 if dtype == "f32" else 4096)
        if kind == "capacity":
            c["factor"] = round(rng.uniform(0.5, 2.0), 2)
        if kind == "mod":
            Bn, S = rng.randint(1, 8), _log(rng, 128, 4096)
            c.update(T=Bn * S, B=Bn, S=S, cap=max(1, int(S * rng.uniform(1 / 16, 1 / 2))))
        if kind == "exit":
            c.update(T=_log(rng, 256, 16384), layers=rng.randint(1, 4), p=round(rng.uniform(0.1, 0.5), 2))
        weights = float(c["H"]) * c["F"] * c.get("E", 1) * c.get("layers", 1)
        if work(c)["flops"] <= MAX_FLOPS[dtype] and weights <= MAX_WEIGHTS:
            return c


def _capacity(c):
    """Rows an expert may take: `factor` times its even share."""
    return max(1, int(c["factor"] * c["T"] * c["k"] / c["E"]))


class State:
    pass


def prepare(case, seed):
    c, s = case, State()
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    act = torch.float32 if c["dtype"] == "f32" else torch.bfloat16

    def normal(shape, sigma=1.0, dtype=act):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, sigma, generator=gen)

    T, H, F, E, L = c["T"], c["H"], c["F"], c.get("E", 1), c.get("layers", 1)
    mode = {"mod": "mod", "exit": "early_exit"}.get(c["kind"], "moe")
    s.case = c
    s.layers = [RoutedFFNLayer(T, H, F, E, c.get("k", 1), c["dtype"], mode) for _ in range(L)]
    s.weights = [(normal((E, F, H), 0.02), normal((E, F, H), 0.02), normal((E, H, F), 0.02)) for _ in range(L)]
    s.x = normal((T, H))
    if c["kind"] != "forward":
        s.dout = normal((T, H))
        for layer in s.layers:
            layer.alloc_backward()
    if mode == "moe":
        zipf = torch.arange(1, E + 1, dtype=torch.float32, device="cuda").pow(-c["zipf"])
        s.logits = normal((T, E), 1.0, torch.float32) + zipf
    elif mode == "mod":
        s.scores = normal((c["B"], c["S"]), 1.0, torch.float32)
    else:
        s.exit_layer = torch.empty(T, dtype=torch.float32, device="cuda").geometric_(c["p"], generator=gen).to(torch.int32)
    if c["kind"] == "capacity":
        d = s.layers[0].d
        s.bias = normal((E,), 0.1, torch.float32)
        s.chosen = torch.empty((T, c["k"]), dtype=torch.int32, device="cuda")
        s.ws_drop = torch.empty(B.dynmo_route_drop_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    return {"moe": _run_moe, "capacity": _run_capacity, "top1": _run_top1, "mod": _run_mod, "exit": _run_exit,
            "forward": _run_forward}[s.case["kind"]](s)


def _grads(layer):
    return {"dWg": layer.dWg, "dWu": layer.dWu, "dWd": layer.dWd}


def _run_moe(s):
    layer, W = s.layers[0], s.weights[0]
    layer.route_topk(s.logits)
    out = layer.forward(s.x, *W)
    layer.load_begin()
    dx = layer.backward(s.dout, *W)
    dlogits = layer.route_bwd()
    counts, load = layer.load_end()
    return {"out": out, "dx": dx, "dlogits": dlogits, "counts": np.asarray(counts), **_grads(layer)}


def _run_capacity(s):
    layer, W, d = s.layers[0], s.weights[0], s.layers[0].d
    B.dynmo_route_topk_ex(d, s.logits, s.bias, B.NORM_ALL, s.chosen, layer.gate_w)
    B.dynmo_route_drop(d, s.chosen, _capacity(s.case), layer.expert_idx, s.ws_drop)
    out = layer.forward(s.x, *W)
    layer.load_begin()
    dx = layer.backward(s.dout, *W)
    B.dynmo_route_topk_all_bwd(d, layer.dgate, s.logits, s.chosen, layer.droute)
    counts, load = layer.load_end()
    return {"out": out, "dx": dx, "dlogits": layer.droute, "kept": layer.expert_idx, "counts": np.asarray(counts), **_grads(layer)}


def _run_top1(s):
    layer, W = s.layers[0], s.weights[0]
    layer.route_topk(s.logits)
    out = layer.forward_folded(s.x, *W)
    layer.load_begin()
    dx = layer.backward_folded(s.dout, *W)
    counts, load = layer.load_end()
    return {"out": out, "dx": dx, "dgate": layer.dgate, "counts": np.asarray(counts), **_grads(layer)}


def _run_mod(s):
    layer, W = s.layers[0], s.weights[0]
    layer.route_capacity(s.scores, s.case["cap"])
    out = layer.forward(s.x, *W)
    layer.load_begin()
    dx = layer.backward(s.dout, *W)
    dscores = layer.route_bwd(s.scores)
    counts, load = layer.load_end()
    return {"out": out, "dx": dx, "dscores": dscores, "selected": layer.expert_idx, "counts": np.asarray(counts), **_grads(layer)}


def _run_exit(s):
    x = s.x
    for i, layer in enumerate(s.layers):
        layer.route_active(s.exit_layer, i + 1)
        x = layer.forward(x, *s.weights[i])
        layer.load_begin()
    g = s.dout
    for i in range(len(s.layers) - 1, -1, -1):
        g = s.layers[i].backward(g, *s.weights[i])
    loads = [layer.load_end()[1] for layer in s.layers]
    if len(loads) > 1:
        B.dynmo_partition(loads, 2)
    return {"out": x, "dx": g, "loads": np.asarray(loads), "grads": [_grads(layer) for layer in s.layers]}


def _run_forward(s):
    layer, W = s.layers[0], s.weights[0]
    layer.route_topk(s.logits)
    out = layer.forward_gather(s.x, *W)
    return {"out": out, "experts": layer.expert_idx, "gates": layer.gate_w}


def _rows(c):
    """Routed rows of each layer (expected where the inputs decide)."""
    if c["kind"] == "mod":
        return [c["B"] * c["cap"]]
    if c["kind"] == "exit":
        return [c["T"] * (1.0 - c["p"]) ** i for i in range(c["layers"])]
    if c["kind"] == "capacity":  # the two most loaded experts overflow first; most rows are kept
        return [min(c["T"] * c["k"], c["E"] * _capacity(c))]
    return [c["T"] * c["k"]]


def work(case):
    c = case
    b = 4 if c["dtype"] == "f32" else 2
    HF, E, rows = float(c["H"]) * c["F"], c.get("E", 1), _rows(c)
    tokens = float(c["T"]) * c["H"] * b
    router = float(c["T"]) * E * 4
    if c["kind"] == "forward":  # x and the weights of the experts in use in, out out
        used = min(E, c["T"] * c["k"])
        return {"bytes": 2 * tokens + 3 * used * HF * b + router, "flops": 6 * HF * rows[0]}
    # x, dout and the weights in; out, dx and the weight gradients out; logits or scores in, their gradient out
    return {"bytes": 4 * tokens + 6 * E * HF * b * len(rows) + 2 * router, "flops": 18 * HF * sum(rows)}


def tolerance(case):
    """About four times the distance of each output to the same step computed in 64 bits (2-norm; largest element)."""
    if case["dtype"] == "f32":  # seen: rel up to 1.0e-6 (K = 1030), largest element 8e-6
        return {"rel": 5e-6, "max": 4e-5}
    if case["kind"] == "exit":  # roundings add up over the layers.  Seen: rel up to 1.2e-2, largest element 0.17
        return {"rel": 3e-2, "max": 0.6}
    return {"rel": 1.5e-2, "max": 0.25}  # seen: rel up to 3.9e-3, largest element 7.1e-2 (experts with few rows)
