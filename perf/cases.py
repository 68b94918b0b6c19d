"""The work that a user of this library has it do, as cases that can be timed and compared.

A case names the layers ("<d_in>x<d_out>k<weak columns>", separated by blanks), how they are quantised and packed,
the number of tokens and which entry point is called:

  path "linear"    OwqLinear(x) on every layer of `blocks` blocks; with graph=True as a serving loop runs it, the calls
                   of one step captured in a HIP graph that is kept and replayed
  path "tasks"     OwqLinear.multi: several task-specific sets of weak columns over one low-bit matrix
  path "backward"  OwqLinear.backward: gradients for weak-column tuning (dX and dWw)
  path "search"    search_config: step sizes, zero points and codes from fp16 weights

Layers follow synth/layers.py's recipe, drawn on the GPU: codes U{0..2^bits-1}, step sizes U(0.001, 0.01), zero points
U{0..2^bits-1}, weak columns N(0, 0.02), activations N(0, 1) with a factor of 20 at the weak columns (the outliers they
are kept in fp16 for), gradients N(0, 0.05).
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2306_02272_amd import binding

GEMV, TILE, COMPACT = binding.OWQ_LAYOUT_GEMV, binding.OWQ_LAYOUT_TILE, binding.OWQ_LAYOUT_COMPACT


def _linear(layers, bits, group, layout, tokens, blocks=1, graph=False):
    return {"path": "linear", "layers": layers, "bits": bits, "group": group, "layout": layout, "tokens": tokens,
            "blocks": blocks, "graph": graph}


def _tasks(layers, bits, group, layout, tokens, sets):
    return {"path": "tasks", "layers": layers, "bits": bits, "group": group, "layout": layout, "tokens": tokens, "sets": sets}


def _backward(layers, bits, group, tokens):
    return {"path": "backward", "layers": layers, "bits": bits, "group": group, "layout": TILE, "tokens": tokens}


def _search(layers, bits, group, grid, shrink):
    return {"path": "search", "layers": layers, "bits": bits, "group": group, "grid": grid, "shrink": shrink}


def listed():
    return [
        # one call on a small layer, launched by itself: what a call costs at least
        dict(_linear("1024x1024k8", 4, 0, GEMV, 1), name="small_call"),
        # a token through the feed-forward pairs of four blocks, 3-bit codes from HBM
        dict(_linear("4096x16384k32 16384x4096k128", 3, 128, GEMV, 1, blocks=4, graph=True), name="decode_1_3bit"),
        # a token through the seven projections of a 4-bit block, twice
        dict(_linear("5120x5120k51 5120x5120k51 5120x5120k51 5120x5120k51 5120x13824k51 5120x13824k51 13824x5120k138",
                     4, 128, GEMV, 1, blocks=2, graph=True), name="decode_1_4bit"),
        # the same block for 16 requests that are decoded together
        dict(_linear("5120x5120k51 5120x5120k51 5120x5120k51 5120x5120k51 5120x13824k51 5120x13824k51 13824x5120k138",
                     4, 128, TILE, 16, blocks=2, graph=True), name="decode_16_4bit"),
        # 64 requests decoded together, the largest feed-forward pair, one scale per row
        dict(_linear("9216x36864k64 36864x9216k256", 3, 0, TILE, 64), name="decode_64_3bit"),
        # a long prompt, or a batch of prompts, through a 3-bit feed-forward pair
        dict(_linear("4096x16384k32 16384x4096k128", 3, 128, TILE, 2048), name="prefill_2048_3bit"),
        # one prompt of a length that is no multiple of anything, 4-bit
        dict(_linear("5120x13824k51 13824x5120k138", 4, 128, TILE, 777), name="prefill_777_4bit"),
        # requests of several tasks in one batch on a layer whose sides are no multiples of a tile
        dict(_tasks("7000x3333k70", 4, 128, TILE, 37, 5), name="tasks_37_ragged"),
        # weak-column tuning: gradients of a feed-forward pair for a micro-batch of 512 tokens
        dict(_backward("4096x16384k32 16384x4096k128", 3, 128, 512), name="backward_512_3bit"),
        # the same for a longer, uneven batch on a 4-bit layer
        dict(_backward("5120x13824k51", 4, 128, 1000), name="backward_1000_4bit"),
        # configuration search when a layer is quantised: one scale per 128 columns
        dict(_search("4096x16384k32", 3, 128, 16, 0.4), name="search_group_3bit"),
        # and one scale per row
        dict(_search("5120x5120k51", 4, 0, 16, 0.4), name="search_row_4bit"),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _side(rng):
    """A layer's side, 512 to 16384: a multiple of 128 mostly, as hidden sizes are, now and then any number."""
    n = _log_int(rng, 512, 16384)
    return n if rng.random() < 0.25 else max(512, n // 128 * 128)


def draw(rng):
    bits, group = rng.choice((3, 4)), rng.choice((0, 128, 128, 256))
    d_in, d_out = _side(rng), _side(rng)
    if d_in * d_out > 1 << 27:
        d_out = max(512, (1 << 27) // d_in)
    layer = "%dx%dk%d" % (d_in, d_out, max(1, round(d_in * rng.uniform(0.004, 0.012))))
    path = rng.choice(("decode", "decode", "batch", "batch", "prefill", "prefill", "tasks", "backward", "backward", "search"))
    if path == "decode":      # single-token layouts: the number of blocks keeps the weights out of the caches, as a model's would be
        blocks = max(1, min(16, (96 << 20) * 8 // (d_in * d_out * bits)))
        if group == 0 and rng.random() < 0.3:
            return _linear(layer, bits, 0, COMPACT, 1, blocks, True)
        return _linear(layer, bits, group, GEMV, rng.choice((1, 1, 1, 2, 3)), blocks, True)
    if path == "batch":
        blocks = max(1, min(8, (96 << 20) * 8 // (d_in * d_out * bits)))
        return _linear(layer, bits, group, TILE, _log_int(rng, 4, 64), blocks, True)
    if path == "prefill":
        return _linear(layer, bits, group, TILE, _log_int(rng, 65, 2048))
    if path == "tasks":
        return _tasks(layer, bits, group, TILE, _log_int(rng, 2, 64), rng.randint(2, 8))
    if path == "backward":
        return _backward(layer, bits, group, _log_int(rng, 16, 1024))
    return _search(layer, bits, group, rng.choice((8, 12, 16)), round(rng.uniform(0.2, 0.45), 3))


class _Spec:
    """A layer in plain form on the host, as the packer takes it."""


def _shapes(case):
    out = []
    for text in case["layers"].split():
        d_in, rest = text.split("x")
        d_out, k = rest.split("k")
        out.append((int(d_in), int(d_out), int(k)))
    return out


def _groups(case, d_in):
    return 1 if case["group"] == 0 else -(-d_in // case["group"])


def _layer(case, d_in, d_out, k, gen):
    """One layer drawn on the GPU and brought to the host."""
    dev = "cuda"
    s = _Spec()
    s.d_in, s.d_out, s.bits, s.group_size, s.k = d_in, d_out, case["bits"], case["group"], k
    levels, groups = 1 << s.bits, _groups(case, d_in)
    idx = torch.randperm(d_in, generator=gen, device=dev)[:k].sort().values
    codes = torch.randint(0, levels, (d_out, d_in), dtype=torch.uint8, generator=gen, device=dev)
    codes[:, idx] = 0
    scale = torch.rand((d_out, groups), generator=gen, device=dev) * 0.009 + 0.001
    zero = torch.randint(0, levels, (d_out, groups), generator=gen, device=dev)
    weak = torch.randn((d_out, k), generator=gen, device=dev) * 0.02
    s.codes, s.weak_idx = codes.cpu().numpy(), idx.to(torch.int32).cpu().numpy()
    s.scale, s.zero = scale.half().cpu().numpy(), zero.half().cpu().numpy()
    s.weak_w = weak.half().cpu().numpy()
    return s, idx


def _activations(tokens, d_in, idx, gen):
    x = torch.randn((tokens, d_in), generator=gen, device="cuda")
    x[:, idx] *= 20.0
    return x.half()


def _prepare_search(case, gen):
    (d_in, d_out, k), = _shapes(case)
    idx = torch.randperm(d_in, generator=gen, device="cuda")[:k].sort().values
    w = torch.randn((d_out, d_in), generator=gen, device="cuda") * 0.02
    # 0.2 % of the entries are a long tail, which a narrowed range cuts off; the weak columns are large
    tail = torch.rand((d_out, d_in), generator=gen, device="cuda") < 0.002
    w = torch.where(tail, w * (3 + 7 * torch.rand((d_out, d_in), generator=gen, device="cuda")), w)
    w[:, idx] *= 6.0
    return {"case": case, "w": w.half(), "idx": idx.to(torch.int32)}


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["path"] == "search":
        return _prepare_search(case, gen)
    layers, lins = {}, []
    for block in range(case.get("blocks", 1)):
        for shape in _shapes(case):
            if shape in layers:       # another layer of this shape, in memory of its own
                spec, idx, first = layers[shape]
                lin = binding.OwqLinear(spec, packed=first.buf, layout=case["layout"])
            else:
                spec, idx = _layer(case, *shape, gen)
                lin = binding.OwqLinear(spec, layout=case["layout"])
                layers[shape] = (spec, idx, lin)
            lins.append((lin, _activations(case["tokens"], shape[0], idx, gen)))
    state = {"case": case, "lins": lins}
    if case["path"] == "backward":
        state["dy"] = [(torch.randn((case["tokens"], lin.d_out), generator=gen, device="cuda") * 0.05).half() for lin, _ in lins]
    elif case["path"] == "tasks":
        (lin, _), = lins
        (_, d_out, k), = _shapes(case)
        sets = [(torch.randn((d_out, k), generator=gen, device="cuda") * 0.02).half().cpu().numpy() for _ in range(case["sets"])]
        state["table"], state["sets"] = lin.add_weak_sets(sets)
        # -1: a request without a task of its own
        state["task"] = torch.randint(-1, case["sets"], (case["tokens"],), dtype=torch.int32, generator=gen, device="cuda")
    elif case["graph"]:
        state["ys"] = [torch.empty((case["tokens"], lin.d_out), dtype=torch.float16, device="cuda") for lin, _ in lins]
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"], stream=stream):
            for (lin, x), y in zip(lins, state["ys"]):
                lin(x, out=y)
    return state


def run(state):
    case = state["case"]
    if case["path"] == "search":
        return binding.search_config(state["w"], state["idx"], case["bits"], case["group"], case["grid"], case["grid"], case["shrink"])
    if case["path"] == "backward":
        return [lin.backward(dy, x) for (lin, x), dy in zip(state["lins"], state["dy"])]
    if case["path"] == "tasks":
        (lin, x), = state["lins"]
        return lin.multi(x, state["table"], state["task"])
    if case["graph"]:
        state["graph"].replay()
        return state["ys"]
    return [lin(x) for lin, x in state["lins"]]


def work(case):
    shapes = _shapes(case) * case.get("blocks", 1)
    nbytes = flops = 0.0
    for d_in, d_out, k in shapes:
        groups = _groups(case, d_in)
        if case["path"] == "search":
            # weights once in; step sizes, zero points, codes, errors and choices once out; the error of one grid
            # point (7 operations a weight): the others need not be summed to the end to be ruled out
            nbytes += 2 * d_out * d_in + 4 * k + d_out * groups * (2 + 2 + 4 + 4) + d_out * d_in
            flops += 7 * d_out * d_in
            continue
        t = case["tokens"]
        cols = d_in - k if case["layout"] == COMPACT else d_in
        nbytes += d_out * cols * case["bits"] / 8 + 4 * d_out * groups + 2 * d_out * k * case.get("sets", 1) + 4 * k
        flops += 2 * t * d_in * d_out
        if case["path"] == "backward":
            nbytes += 2 * t * (d_out + k) + 2 * t * d_in + 4 * d_out * k
            flops += 2 * t * k * d_out
        else:
            nbytes += 2 * t * (d_in + d_out)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["path"] == "search":
        # every operation that decides a step size, zero point or code is one binary32 operation; only grid points whose
        # errors agree to the rounding of their binary32 sums (1e-5 of 5120 terms) may be exchanged (none of 2304 were)
        return {"rel": 2e-3, "max": 0.99, "differ": 1e-4}
    if case["path"] == "backward":
        # dX against the product in 64 bits: 2.9e-4, at most 1.3e-3 (dY times the step size and dX are rounded to fp16)
        return {"rel": 1.2e-3, "max": 5.5e-3}
    # against the product in 64 bits: 2.1e-4, at most 6.6e-4 (the one rounding of y to fp16)
    return {"rel": 9e-4, "max": 3e-3}
