"""The work a user of the library has it do, as cases that can be timed and compared.

Every case goes through the public entry points (``paper_2511_15015_amd.binding.Context`` and the caller-side
glue of ``paper_2511_15015_amd.layer``) on synthetic inputs of the shapes that ``workloads.py`` names:
activations N(0, 1), weights N(0, 0.02), router logits with the spread of x . W_r for such a router plus a Zipf
bias under a permutation of its own per layer, and the experts with the largest bias resident in the pair's
high format (what the top-n selection of the router traces arrives at).

Kinds of cases:

``layer``   one ``dx_route_forward`` call per layer (routing, hotness counters, expert execution, combine), the
            layers one after the other with weights of their own, as a decode step or a prefill chunk runs
            them.  Few tokens mean several layers, so that the weights of a pass do not sit in the last-level
            cache from the pass before.
``router``  one ``dx_router_logits`` call per layer.
``quantize`` the low-precision versions of a number of experts, one launch per matrix kind, as the set-up of a
            layer and a window's demotions make them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2511_15015_amd import binding as B
from paper_2511_15015_amd import layer as LY

# model shapes of workloads.py: experts, top-k, hidden size, expert intermediate size, always-resident shared
# expert, experts in the high format, Zipf exponent of the router's skew
SHAPES = {
    "30b": dict(E=128, k=8, d=2048, f=768, shared_f=0, n_hi=32, zipf=1.1),
    "80b": dict(E=512, k=10, d=2048, f=512, shared_f=512, n_hi=12, zipf=1.0),
    "phi": dict(E=16, k=2, d=4096, f=6400, shared_f=0, n_hi=4, zipf=1.0),
}


def _layer(name, shape, T, layers, pair="bf16-int4", group=128):
    return {"name": name, "kind": "layer", "shape": shape, "T": T, "layers": layers, "pair": pair, "group": group}


def listed():
    return [
        # one sequence being decoded: latency and launches
        _layer("decode_1_30b", "30b", 1, 8),
        # the batch of 32 that the benchmark decodes, both model shapes (the second: many experts, most of them
        # int4, and a shared expert)
        _layer("decode_32_30b", "30b", 32, 4),
        _layer("decode_32_80b", "80b", 32, 4),
        # an odd decode batch on the quantized precision pair, groups of 64
        _layer("decode_17_30b_int4_int2", "30b", 17, 4, "int4-int2", 64),
        # a large or speculative decode batch, no multiple of anything
        _layer("decode_101_30b", "30b", 101, 2),
        # a short prompt or a chunk of one
        _layer("prefill_300_30b", "30b", 300, 2),
        # prompts on the many-expert shape: short segments, a long shared one
        _layer("prefill_1000_80b", "80b", 1000, 2),
        # few, very large experts
        _layer("prefill_1100_phi", "phi", 1100, 1),
        # the prefill batch of the benchmark
        _layer("prefill_4096_30b", "30b", 4096, 1),
        # the router's gate in front of the layer: a decode step's, and a prefill chunk's
        {"name": "router_32_80b", "kind": "router", "shape": "80b", "T": 32, "layers": 8, "bias": False},
        {"name": "router_4096_30b", "kind": "router", "shape": "30b", "T": 4096, "layers": 2, "bias": True},
        # demotions of a window, or the set-up of a layer's low tier
        {"name": "quantize_48_30b", "kind": "quantize", "shape": "30b", "experts": 48, "bits": 4, "group": 128},
    ]


def draw(rng):
    kind = rng.choice(["layer"] * 7 + ["router"] * 2 + ["quantize"])
    if kind == "quantize":
        bits = rng.choice([4, 4, 2])
        return {"kind": kind, "shape": rng.choice(["30b", "80b"]), "experts": round(math.exp(rng.uniform(0, math.log(96)))),
                "bits": bits, "group": rng.choice([64, 128] if bits == 2 else [32, 64, 128, 128])}
    if kind == "router":
        return {"kind": kind, "shape": rng.choice(["30b", "80b", "phi"]), "T": round(math.exp(rng.uniform(0, math.log(4096)))),
                "layers": rng.choice([1, 2, 4]), "bias": rng.random() < 0.5}
    shape = rng.choice(["30b", "30b", "30b", "80b", "80b", "phi"])
    T = round(math.exp(rng.uniform(0, math.log({"30b": 4096, "80b": 3000, "phi": 1100}[shape]))))
    return {"kind": kind, "shape": shape, "T": T, "layers": 1 if shape == "phi" or T > 128 else 4 if T > 2 else 8,
            "pair": "bf16-int4" if shape == "80b" else rng.choice(["bf16-int4", "bf16-int4", "int4-int2"]),
            "group": rng.choice([128, 128, 128, 64])}


# ---- inputs, from the seed alone ------------------------------------------------------------------------------
def _generator(seed, layer, what):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + layer * 101 + what) & 0x7FFFFFFFFFFF)
    return g


def _randn(g, shape, std=1.0):
    t = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    return t.mul_(std).to(torch.bfloat16)


def _zipf_bias(s, seed, layer):
    z = np.arange(1, s["E"] + 1, dtype=np.float64) ** -s["zipf"]
    return np.log(z / z.sum())[np.random.default_rng([seed & 0x7FFFFFFF, layer]).permutation(s["E"])].astype(np.float32)


def _layer_inputs(case, seed, layer):
    """x [T,d] bf16 and logits [T,E] fp32 on the device; the ids in the high format."""
    s = SHAPES[case["shape"]]
    x = _randn(_generator(seed, layer, 0), (case["T"], s["d"]))
    bias = _zipf_bias(s, seed, layer)
    noise = torch.randn((case["T"], s["E"]), generator=_generator(seed, layer, 1), device="cuda", dtype=torch.float32)
    logits = noise * (0.02 * math.sqrt(s["d"])) + torch.from_numpy(bias).cuda()
    return x, logits, np.argsort(-bias, kind="stable")[: s["n_hi"]]


def _masters(case, seed, layer):
    """bf16 masters of the routed experts: gate [E,f,d], up [E,f,d], down [E,d,f]."""
    s = SHAPES[case["shape"]]
    g = _generator(seed, layer, 2)
    return [_randn(g, sh, 0.02) for sh in ((s["E"], s["f"], s["d"]), (s["E"], s["f"], s["d"]), (s["E"], s["d"], s["f"]))]


def _shared(case, seed, layer):
    s = SHAPES[case["shape"]]
    g = _generator(seed, layer, 3)
    return [_randn(g, sh, 0.02) for sh in ((s["shared_f"], s["d"]), (s["shared_f"], s["d"]), (s["d"], s["shared_f"]))]


def _router_inputs(case, seed, layer):
    s = SHAPES[case["shape"]]
    g = _generator(seed, layer, 4)
    x, w = _randn(g, (case["T"], s["d"])), _randn(g, (s["E"], s["d"]), 0.02)
    return x, w, torch.from_numpy(_zipf_bias(s, seed, layer)).cuda() if case["bias"] else None


def _quantize_inputs(case, seed):
    s = SHAPES[case["shape"]]
    g, n = _generator(seed, 0, 5), case["experts"]
    return [_randn(g, sh, 0.02) for sh in ((n * s["f"], s["d"]), (n * s["f"], s["d"]), (n * s["d"], s["f"]))]


# ---- what a program has in hand before the call ----------------------------------------------------------------
def _context(case, **kw):
    s = SHAPES[case["shape"]]
    return B.Context(E=s["E"], d=s["d"], f=s["f"], top_k=s["k"], shared_f=s["shared_f"], **kw)


def prepare(case, seed):
    s = SHAPES[case["shape"]]
    if case["kind"] == "quantize":
        ctx = _context(case, L=1, group=case["group"], max_tokens=1)
        src = _quantize_inputs(case, seed)
        per = 8 // case["bits"]
        out = [(torch.empty((m.shape[0], m.shape[1] // per), dtype=torch.uint8, device="cuda"),
                torch.empty((m.shape[0], m.shape[1] // case["group"]), dtype=torch.bfloat16, device="cuda")) for m in src]
        return {"case": case, "ctx": ctx, "src": src, "out": out}
    L, T = case["layers"], case["T"]
    if case["kind"] == "router":
        ctx = _context(case, L=L, group=128, max_tokens=T)
        ins = [_router_inputs(case, seed, layer) for layer in range(L)]
        return {"case": case, "ctx": ctx, "in": ins,
                "logits": [torch.empty((T, s["E"]), dtype=torch.float32, device="cuda") for _ in range(L)]}
    quantized = case["pair"] == "int4-int2"
    ctx = _context(case, L=L, group=case["group"], max_tokens=T, route_updates_hotness=True,
                   hi_fmt=B.DX_FMT_INT4G if quantized else B.DX_FMT_BF16)
    state = {"case": case, "ctx": ctx, "x": [], "logits": [], "weights": [], "shared": [], "rb": [], "y": []}
    for layer in range(L):
        x, logits, hi = _layer_inputs(case, seed, layer)
        wg, wu, wd = _masters(case, seed, layer)
        if quantized:
            weights = LY.QuantPairLayerWeights(ctx, layer, wg, wu, wd, hi, case["group"])
        else:
            weights = LY.LayerWeights(ctx, layer, wg, wu, wd, hi, case["group"], keep_masters=False)
        del wg, wu, wd
        if s["shared_f"]:
            state["shared"].append(_shared(case, seed, layer))
            ctx.dx_swap_handle(layer, s["E"], B.make_handle(B.DX_FMT_BF16, *state["shared"][layer]))
        state["x"].append(x)
        state["logits"].append(logits)
        state["weights"].append(weights)
        state["rb"].append(LY.RoutingBuffers(T, s["E"], s["k"]))
        state["y"].append(torch.empty((T, s["d"]), dtype=torch.bfloat16, device="cuda"))
    return state


def run(state):
    case, ctx = state["case"], state["ctx"]
    if case["kind"] == "quantize":
        quantize = ctx.dx_quantize_expert if case["bits"] == 4 else ctx.dx_quantize_expert_int2
        for m, (q, sc) in zip(state["src"], state["out"]):
            quantize(m, m.shape[0], m.shape[1], case["group"], q, sc)
        return state["out"]
    if case["kind"] == "router":
        for (x, w, bias), logits in zip(state["in"], state["logits"]):
            ctx.dx_router_logits(x, w, bias, case["T"], logits)
        return state["logits"]
    for layer in range(case["layers"]):
        state["rb"][layer].route_forward(ctx, layer, state["logits"][layer], state["x"][layer], state["y"][layer])
    return [(y, rb.ids, rb.w, rb.counts, rb.offsets, rb.perm) for y, rb in zip(state["y"], state["rb"])]


# ---- what a pass cannot do without -----------------------------------------------------------------------------
def _version_bytes(s, group, fmt):
    n = 3 * s["d"] * s["f"]
    return 2 * n if fmt == "bf16" else n // (2 if fmt == "int4" else 4) + 2 * n // group


def work(case):
    s = SHAPES[case["shape"]]
    if case["kind"] == "quantize":
        n = 3 * case["experts"] * s["d"] * s["f"]
        return {"bytes": n * (2 + case["bits"] / 8) + 2 * n / case["group"], "flops": 0}
    T, E, k, d, f, L = case["T"], s["E"], s["k"], s["d"], s["f"], case["layers"]
    if case["kind"] == "router":
        return {"bytes": L * (2 * T * d + 2 * E * d + 4 * T * E + (4 * E if case["bias"] else 0)), "flops": L * 2 * T * E * d}
    hi, lo = case["pair"].split("-")
    total = flops = 0
    for layer in range(L):
        # the experts that tokens of this skew select: one draw of the same distribution (on the CPU)
        rng = np.random.default_rng([7, layer])
        bias = _zipf_bias(s, 7, layer)
        logits = rng.standard_normal((T, E), dtype=np.float32) * (0.02 * math.sqrt(d)) + bias
        active = np.unique(np.argpartition(-logits, k - 1, axis=1)[:, :k])
        n_hi = int(np.isin(active, np.argsort(-bias, kind="stable")[: s["n_hi"]]).sum())
        total += n_hi * _version_bytes(s, case["group"], hi) + (len(active) - n_hi) * _version_bytes(s, case["group"], lo)
        total += 6 * d * s["shared_f"]
        # x and y, logits, ids and weights and permutation, counts and offsets
        total += 4 * T * d + 4 * T * E + 12 * T * k + 8 * E
        flops += 6 * T * d * (k * f + s["shared_f"])
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["kind"] == "quantize":
        return "exact"
    if case["kind"] == "router":
        # fp32 sums of 2048 to 4096 bf16 products: 2e-7 and 9e-7 measured against 64 bits, times four
        return {"rel": 8e-7, "max": 4e-6}
    # H and y (and, above 128 tokens, the experts' outputs) are stored in bf16: up to 3.1e-3 and 1.8e-2 measured
    # against 64 bits, times about four; routing is exact
    return {"rel": 1e-2, "max": 6e-2, "differ": 0.0}


# ---- the same in 64 bits, without the library -------------------------------------------------------------------
def _dequantized(w, group, fmt):
    """Values of the stored version, 64 bits (the rule's own decisions are taken in fp32)."""
    if fmt == "bf16":
        return w.double()
    qmax = 7.0 if fmt == "int4" else 1.0
    g = w.float().reshape(w.shape[0], -1, group)
    scale = (g.abs().amax(-1, keepdim=True) / qmax).to(torch.bfloat16).float()
    q = torch.where(scale > 0, torch.clamp(torch.round(g / scale), -qmax - 1, qmax), torch.zeros_like(g))
    return (q.double() * scale.double()).reshape(w.shape)


def _swiglu(x, wg, wu, wd):
    g = x @ wg.t()
    return (g * torch.sigmoid(g) * (x @ wu.t())) @ wd.t()


def exact(case, seed):
    s = SHAPES[case["shape"]]
    if case["kind"] == "quantize":
        qmax = 7.0 if case["bits"] == 4 else 1.0
        return [(None, m.double().abs().reshape(m.shape[0], -1, case["group"]).amax(-1) / qmax) for m in _quantize_inputs(case, seed)]
    if case["kind"] == "router":
        out = []
        for layer in range(case["layers"]):
            x, w, bias = _router_inputs(case, seed, layer)
            out.append(x.double() @ w.double().t() + (bias.double() if bias is not None else 0.0))
        return out
    hi_fmt, lo_fmt = case["pair"].split("-")
    out = []
    for layer in range(case["layers"]):
        x, logits, hi = _layer_inputs(case, seed, layer)
        masters = _masters(case, seed, layer)
        top, ids = torch.sort(logits.double(), dim=1, descending=True, stable=True)
        ids, w = ids[:, : s["k"]], torch.softmax(top[:, : s["k"]], dim=1)
        xd = x.double()
        y = torch.zeros((case["T"], s["d"]), dtype=torch.float64, device="cuda")
        for e in torch.unique(ids).tolist():
            tok, slot = torch.nonzero(ids == e, as_tuple=True)
            wg, wu, wd = (_dequantized(m[e], case["group"], hi_fmt if e in hi else lo_fmt) for m in masters)
            y.index_add_(0, tok, w[tok, slot, None] * _swiglu(xd[tok], wg, wu, wd))
        if s["shared_f"]:
            y += _swiglu(xd, *(m.double() for m in _shared(case, seed, layer)))
        out.append((y, None, w, None, None, None))
    return out
