"""What the layer's speed is measured on: its calls as programs make them, over their range.

A case is one forward pass of MoEShardLayer (routing, grouping, expert step, combine) on a
batch of T tokens, or ("load") loadShard followed by such a pass.  listed() holds the shapes
of this repository's workloads (synth/workloads.py) and generic ones beside them: decode
batches, prompts, ragged sizes, both data types, the three activations, top-1 and top-2,
fp32 shard partials.  draw() gives others of the same ranges.

Fields of a case: T tokens, h hidden size, E experts, k picks, F full inner width, f the
shard's inner width (columns [col0, col0 + f)), act, dtype ("bf16" / "f32"), out ("same", or
"f32": y_perm and y as unrounded fp32 partials, which another device's would be added to),
routing, renorm, load (whether the shard is packed inside the pass).

Routing kinds, as in synth/workloads.py: "gate" (logits only), "shared" (one selection bias
per expert, as load balancing without an auxiliary loss keeps), and per-token target sets
drawn from "uniform", "zipf" (exponent a), "paper" (b skewed experts, each with probability
1/E + a before normalisation) or "pair" (a fraction a of the tokens on one hot pair): every
target gets a selection bias of 32, above the spread of the logits.
"""
from __future__ import annotations

import math

import torch

import paper_2503_08467_amd as moe

BIAS = 32.0
_BASE = dict(T=64, h=1024, E=64, k=2, F=4096, f=4096, col0=0, act="gelu", dtype="bf16", out="same", routing="uniform",
             a=0.0, b=0, renorm=1, load=False)


def _case(name, **kw):
    return dict(_BASE, name=name, **kw)


def listed():
    return [
        # smallest calls: a few sequences decoding on one device's 1/8 shard of a top-2 SwiGLU layer
        _case("decode_4_swiglu", T=4, h=4096, E=8, F=14336, f=1792, act="swiglu", routing="gate"),
        # decode batch of a top-2 layer whose tokens crowd on one expert pair
        _case("decode_64_pair", T=64, routing="pair", a=0.95),
        # one decode step of the 250-sequence batch on a 1/4 shard of a 128-expert top-1 layer
        _case("decode_250_top1", T=250, h=768, E=128, k=1, F=3072, f=768, routing="paper", a=0.6, b=13, renorm=0),
        # small fp32 layer, full experts, the gate alone decides
        _case("small_f32", T=512, h=768, E=8, k=1, F=3072, f=3072, dtype="f32", routing="gate", renorm=0),
        # nothing a multiple of a tile: odd token count, hidden size a multiple of 8 only, an odd
        # shard of the inner width, the tanh form of GELU
        _case("ragged_tanh", T=1531, h=776, E=24, F=4095, f=1365, col0=1365, act="gelu_tanh"),
        # a layer whose shard is cut out of the full weights for this pass, then used for a prompt
        _case("load_prefill", T=2048, E=32, f=1024, col0=1024, load=True),
        # fp32 partial outputs of a 1/8 shard, to be summed over the devices
        _case("partial_f32", T=4096, f=512, col0=512, out="f32", routing="zipf", a=1.0),
        # prompts on a Switch-sized top-1 layer, Zipf popularity
        _case("prefill_8k_zipf", T=8192, h=768, k=1, F=3072, f=3072, routing="zipf", a=1.0, renorm=0),
        # prompts on one device's shard of the top-2 SwiGLU layer
        _case("prefill_4k_swiglu", T=4096, h=4096, E=8, F=14336, f=1792, act="swiglu", routing="zipf", a=1.2),
        # 250 sequences of 120 tokens on a 1/4 shard of the 128-expert layer
        _case("prefill_30k_top1", T=30000, h=768, E=128, k=1, F=3072, f=768, routing="paper", a=0.6, b=13, renorm=0),
        # an fp32 prompt batch
        _case("prefill_4k_f32", T=4096, E=16, F=2048, f=2048, dtype="f32"),
        # the largest: 32 768 tokens, full experts, 95 % of the tokens on one expert pair
        _case("prefill_32k_pair", T=32768, routing="pair", a=0.95),
    ]


# No drawn case costs more than the largest listed one: 1.1 TFLOP in bf16 (fp32 products are
# priced 16 times), 1.1 GB of weights.
_MOST_FLOPS, _MOST_WEIGHTS = 1.0e12, 1.0e9


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        act = rng.choice(["gelu", "gelu", "swiglu", "gelu_tanh"])
        T = _log_int(rng, 1, 8192 if dtype == "f32" else 32768)
        E = rng.choice([4, 8, 16, 24, 32, 60, 64, 96, 128])
        k = rng.choice([1, 1, 2, 2, 2, 4])
        # hidden sizes are multiples of 64 in most models; some are multiples of 8 only
        h = 64 * _log_int(rng, 8, 64) if rng.random() < 0.8 else 8 * _log_int(rng, 64, 512)
        # a shard of the inner width: a power-of-two share of a round width, or whatever is left over
        F = 64 * _log_int(rng, 8, 224)
        G = rng.choice([1, 2, 4, 8])
        f = F // G if rng.random() < 0.8 else max(64, F // G - rng.randrange(64))
        out = "f32" if dtype == "bf16" and rng.random() < 0.15 else "same"
        kinds = ["uniform", "zipf", "paper"] + (["pair"] if k == 2 else []) + (["gate", "shared"] if T <= 1024 else [])
        routing = rng.choice(kinds)
        a = {"zipf": rng.choice([0.8, 1.0, 1.2]), "paper": rng.choice([0.3, 0.6]), "pair": rng.choice([0.5, 0.95])}.get(routing, 0.0)
        b = max(1, E // 10) if routing == "paper" else 0
        load = rng.random() < 0.08
        c = dict(T=T, h=h, E=E, k=k, F=F, f=f, col0=F - f if rng.random() < 0.5 else 0, act=act, dtype=dtype, out=out,
                 routing=routing, a=a, b=b, renorm=int(k > 1), load=load)
        es, nm = (4, 16) if dtype == "f32" else (2, 1)
        full = _mats(c) * E * h * (F if load else f) * es
        if work(c)["flops"] * nm <= _MOST_FLOPS and full <= _MOST_WEIGHTS:
            return c


def _mats(c):
    return 3 if c["act"] == "swiglu" else 2


def _probabilities(c, device="cpu"):
    """Popularity of the experts, most popular first (float64)."""
    E = c["E"]
    p = torch.full((E,), 1.0 / E, dtype=torch.float64, device=device)
    if c["routing"] == "zipf":
        p = 1.0 / torch.arange(1, E + 1, dtype=torch.float64, device=device) ** c["a"]
    elif c["routing"] == "paper":
        p[: c["b"]] += c["a"]
    return p / p.sum()


def _targets(c, g):
    """k distinct target experts for every token, [T, k]."""
    dev, T, E, k = g.device, c["T"], c["E"], c["k"]
    ids = torch.randperm(E, generator=g, device=dev)
    u = torch.rand((T, E), generator=g, device=dev, dtype=torch.float64).clamp_min_(1e-300)
    # exponential races: the k first arrivals are k draws without replacement
    first = (-torch.log(u) / _probabilities(c, dev)).topk(k, dim=1, largest=False).indices
    tg = ids[first]
    if c["routing"] == "pair":
        hot = torch.rand((T,), generator=g, device=dev) < c["a"]
        tg = torch.where(hot[:, None], ids[:2][None, :], tg)
    return tg


def _inputs(c, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    T, h, E, F = c["T"], c["h"], c["E"], c["F"]
    W = F if c["load"] else c["f"]  # weights outside the shard are there only where the pass cuts it out
    std = 0.01 if h >= 4096 else 0.02

    def normal(shape, s):
        return torch.randn(shape, generator=g, device="cuda", dtype=dt).mul_(s)

    v = {"x": normal((T, h), 1.0), "wg": normal((E, h), std), "w1": normal((E, h, W), std),
         "w3": normal((E, h, W), std) if c["act"] == "swiglu" else None, "w2": normal((E, W, h), std), "bias": None,
         "col0": c["col0"] if c["load"] else 0}
    if c["routing"] == "shared":
        v["bias"] = torch.randn((E,), generator=g, device="cuda").mul_(0.3)
    elif c["routing"] != "gate":
        v["bias"] = torch.zeros((T, E), device="cuda").scatter_(1, _targets(c, g), BIAS)
    return v


def _layer(c, wg, packed):
    out = torch.float32 if c["out"] == "f32" else None
    return moe.MoEShardLayer(wg, packed, c["k"], renorm=bool(c["renorm"]), max_tokens=c["T"], out_dtype=out, partial_dtype=out)


def prepare(case, seed):
    c, v = case, _inputs(case, seed)
    if c["load"]:
        return {"case": c, **v}
    packed = moe.pack_weights(v["w1"], v["w2"], v["w3"], v["col0"], c["f"], act=c["act"])
    return {"case": c, "layer": _layer(c, v["wg"], packed), "x": v["x"], "bias": v["bias"]}


def run(state):
    c = state["case"]
    layer = state.get("layer")
    if layer is None:
        packed = moe.pack_weights(state["w1"], state["w2"], state["w3"], state["col0"], c["f"], act=c["act"])
        layer = _layer(c, state["wg"], packed)
    return layer(state["x"], state["bias"])


def work(case):
    """One pass: activations, gate, selection bias and the weights of the experts that are
    expected to have tokens, read once, and y written once; the products' operations."""
    c = case
    es, ys = (4, 4) if c["dtype"] == "f32" else (2, 4 if c["out"] == "f32" else 2)
    T, h, E, k, f = c["T"], c["h"], c["E"], c["k"], c["f"]
    p = _probabilities(c)
    pick = (1.0 - (1.0 - p) ** k).clamp(max=1.0)  # chance that a token picks the expert
    if c["routing"] == "pair":
        pick = (1.0 - c["a"]) * pick
        pick[:2] += c["a"]
    touched = float((1.0 - (1.0 - pick) ** T).sum())
    bias = {"gate": 0, "shared": 4 * E}.get(c["routing"], 4 * T * E)
    matrices = _mats(c) * h * f * es
    if c["load"]:  # the shard's slices read from the full weights, and the packed shard written
        weights = 2.0 * E * matrices
    else:
        weights = touched * matrices
    return {"bytes": T * h * es + E * h * es + bias + weights + T * h * ys,
            "flops": 2.0 * _mats(c) * T * k * h * f + 2.0 * T * h * E}


def tolerance(case):
    # Four times the largest error of the present path against exact() over the listed and 24
    # drawn cases.  bf16 rounds H, y_perm and y to 8 bits (2.9e-3 at most); rows of a top-1
    # layer without renormalisation differ in scale, so single values are further off (5.7e-2
    # of the root mean square, 1.7e-2 elsewhere).  fp32 sums h and f products (1.2e-6, 8.2e-6).
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 4e-5}
    return {"rel": 1.2e-2, "max": 7e-2 if case["renorm"] else 2e-1}


def exact(case, seed):
    """The layer in 64 bits."""
    c, v = case, _inputs(case, seed)
    if 2.0 * _mats(c) * c["T"] * c["k"] * c["h"] * c["f"] > 2e12:
        return None
    x, T, k = v["x"].double(), c["T"], c["k"]
    logits = x @ v["wg"].double().t()
    scores = logits if v["bias"] is None else logits + v["bias"].double()
    idx = scores.topk(k, dim=1).indices
    w = torch.softmax(logits, dim=1).gather(1, idx)
    if c["renorm"]:
        w = w / w.sum(dim=1, keepdim=True)
    lo, hi = v["col0"], v["col0"] + c["f"]
    y = torch.zeros((T, c["h"]), dtype=torch.float64, device=x.device)
    for e in range(c["E"]):
        t, j = (idx == e).nonzero(as_tuple=True)
        if not t.numel():
            continue
        u = x[t] @ v["w1"][e, :, lo:hi].double()
        if c["act"] == "swiglu":
            u = torch.nn.functional.silu(u) * (x[t] @ v["w3"][e, :, lo:hi].double())
        else:
            u = torch.nn.functional.gelu(u, approximate="tanh" if c["act"] == "gelu_tanh" else "none")
        y.index_add_(0, t, (u @ v["w2"][e, lo:hi].double()) * w[t, j][:, None])
    return y
