"""Timed cases of the activation-sparse FFN forward pass: the calls a decode server makes.

A case names the weights' format, the number of tokens, the layer's shape and the options of
one forward call.  ``listed()`` holds the named cases, ``draw(rng)`` gives others from the same
ranges.  ``prepare`` makes a layer's weights, tokens and workspace, as a server holds them
before a call; ``run`` is one call of the public entry points; ``exact`` is the same call in
64-bit torch.

Keys of a case:
  weights   "f32", "bf16", "i8", "i4"
  tokens    tokens of the call
  d, d_ff   model width and hidden neurons
  r         LoPA rank, 0 for a standard gate
  sparsity  share of inactive neurons of one token
  full      the full form: R-S+ activation, SiLU on W_up and, with LoPA, G and RMSNorm
  dense     every neuron evaluated (the call that a layer takes before it is made sparse)
"""
import math
from statistics import NormalDist

import torch

from paper_2609_31975_amd import ffn

# elements of a 16-byte chunk: real widths and ranks are whole chunks
CHUNK = {"f32": 4, "bf16": 8, "i8": 16, "i4": 32}
WDTYPE_BYTES = {"f32": 4.0, "bf16": 2.0, "i8": 1.0, "i4": 0.5}
QMAX = {"i8": 127, "i4": 7}
RMS_EPS = 1e-6


def _case(weights, tokens, d, d_ff, r, sparsity=0.9, full=False, dense=False):
    return dict(weights=weights, tokens=tokens, d=d, d_ff=d_ff, r=r, sparsity=sparsity, full=full, dense=dense)


def listed():
    named = {
        # the smallest layer: launches and the host side are all there is
        "tiny_f32_std_T1": _case("f32", 1, 256, 1024, 0),
        # one user, one token of an 8B-shaped layer: a gate that is read whole, then the active rows
        "8b_bf16_std_T1": _case("bf16", 1, 4096, 14336, 0),
        # the same layer with a low-rank gate
        "8b_bf16_lopa512_T1": _case("bf16", 1, 4096, 14336, 512),
        # the paper's largest ladder model (level 13, alpha = 1/8) in its own precision; an odd d_ff
        "l13_f32_lopa480_T1": _case("f32", 1, 3840, 14231, 480),
        # weight-only int4 for one user, a standard gate
        "8b_i4_std_T1": _case("i4", 1, 4096, 14336, 0),
        # weight-only int8, a few users (or a few speculated tokens) at once
        "8b_i8_lopa512_T4": _case("i8", 4, 4096, 14336, 512),
        # a small serving batch of the full form
        "8b_bf16_lopa512_full_T16": _case("bf16", 16, 4096, 14336, 512, full=True),
        # a full serving batch
        "8b_bf16_lopa512_T64": _case("bf16", 64, 4096, 14336, 512),
        # a prompt's chunk or a large batch, not a multiple of anything
        "8b_bf16_lopa512_T200": _case("bf16", 200, 4096, 14336, 512),
        # the paper's model and precision for a small batch
        "l13_f32_lopa480_T16": _case("f32", 16, 3840, 14231, 480),
        # the largest layer, one token: the headline workload
        "70b_bf16_std_T1": _case("bf16", 1, 8192, 28672, 0),
        # the largest layer, a few users
        "70b_bf16_lopa1024_T8": _case("bf16", 8, 8192, 28672, 1024),
    }
    return [dict(c, name=n) for n, c in named.items()]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """Another layer: widths over the ladder from tiny to 70B, any d_ff, any batch to 200 tokens."""
    while True:
        weights = rng.choice(["f32", "bf16", "bf16", "i8", "i4"])
        q = CHUNK[weights]
        d = max(256, round(_log_uniform(rng, 256, 8192) / q) * q)
        d_ff = int(d * rng.uniform(2.5, 4.0))
        tokens = 1 if rng.random() < 0.35 else int(_log_uniform(rng, 2, 201))
        r = 0 if rng.random() < 0.4 else max(q, round(d * rng.uniform(0.06, 0.25) / q) * q)
        c = _case(weights, tokens, d, d_ff, r, round(rng.uniform(0.5, 0.97), 3), rng.random() < 0.25,
                  rng.random() < 0.1)
        # no dearer than the listed ones: weights times the passes over them
        if weights == "f32":
            fits = tokens * d * d_ff <= 16 * 3840 * 14231
        elif tokens > 1:
            fits = math.ceil(tokens / 64) * d * d_ff <= 4 * 4096 * 14336
        else:
            fits = True
        if fits:
            return c


def _threshold(case):
    """The gate is close to N(0, 1), with G to N(0, 2)."""
    t = NormalDist().inv_cdf(case["sparsity"])
    return t * math.sqrt(2.0) if case["full"] and case["r"] else t


def _matrix(gen, weights, rows, cols, std):
    """(weights as the entry points take them, fp32 row scales or None)."""
    w = torch.randn((rows, cols), generator=gen, device="cuda")
    if weights in QMAX:
        top = QMAX[weights]
        codes = (w * (top / 3)).round_().clamp_(-top, top).to(torch.int8)
        scale = (0.8 + 0.4 * torch.rand(rows, generator=gen, device="cuda")) * (std / (top / 3))
        if weights == "i4":  # element 2k in the low nibble of byte k
            nib = codes.view(torch.uint8) & 15
            codes = nib[:, 0::2] | (nib[:, 1::2] << 4)
        return codes.contiguous(), scale
    w *= std
    return (w if weights == "f32" else w.to(torch.bfloat16)), None


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    T, d, d_ff, r, weights = case["tokens"], case["d"], case["d_ff"], case["r"], case["weights"]
    s = dict(case, t=_threshold(case))
    s["x"] = torch.randn((T, d), generator=gen, device="cuda")
    names = [("gate", d_ff, r, r ** -0.5), ("lopa_a", r, d, d ** -0.5)] if r else [("gate", d_ff, d, d ** -0.5)]
    scales = {}
    for name, rows, cols, std in names + [("up", d_ff, d, d ** -0.5), ("down", d_ff, d, d_ff ** -0.5)]:
        s[name], scale = _matrix(gen, weights, rows, cols, std)
        if scale is not None:
            scales["lopa_b" if name == "gate" and r else name] = scale
    s["scales"] = scales
    s["sc"] = ffn.scales(**scales) if scales else None
    s["opt"] = None
    if case["full"]:
        lopa = {}
        if r:
            lopa = dict(g_idx=torch.randint(0, d, (d_ff,), generator=gen, device="cuda", dtype=torch.int32),
                        g_sign=(torch.randint(0, 2, (d_ff,), generator=gen, device="cuda") * 2 - 1).to(torch.int8),
                        rms_norm=True, rms_gain=1 + 0.25 * torch.randn(r, generator=gen, device="cuda"),
                        rms_eps=RMS_EPS)
        s["form"] = lopa
        s["opt"] = ffn.options(act=ffn.FFN_ACT_RSPLUS, silu_up=True, **lopa)
    s["y"] = torch.empty((T, d), device="cuda")
    s["ws"] = ffn.alloc_workspace(T, d, d_ff, r)
    kind = "dense" if case["dense"] else "sparse"
    suffix = "_q" if scales else "_ex" if case["full"] else ""
    s["call"] = getattr(ffn, f"ffn_{'lopa_' if r else ''}{kind}_forward{suffix}")
    return s


def run(s):
    gates = (s["lopa_a"], s["gate"]) if s["r"] else (s["gate"],)
    extra = ()
    if s["sc"] is not None:
        return s["call"](s["x"], *gates, s["up"], s["down"], s["sc"], s["t"], s["opt"], s["y"], s["ws"])
    if s["opt"] is not None:
        extra = (s["opt"],)
    return s["call"](s["x"], *gates, s["up"], s["down"], s["t"], *extra, s["y"], s["ws"])


def work(case):
    """Weights read once (the union's rows), tokens in, outputs out; a token's own products only."""
    T, d, d_ff, r = case["tokens"], case["d"], case["d_ff"], case["r"]
    on = 1.0 if case["dense"] else 1.0 - case["sparsity"]
    union = 1.0 - (1.0 - on) ** T
    gate = r * (d + d_ff) if r else d * d_ff
    wb = WDTYPE_BYTES[case["weights"]]
    n = wb * (gate + 2 * union * d_ff * d) + 8.0 * T * d
    if case["weights"] in QMAX:
        n += 4.0 * ((r + d_ff) if r else d_ff) + 8.0 * union * d_ff
    if case["full"] and r:
        n += 5.0 * d_ff + 4.0 * r
    return {"bytes": n, "flops": 2.0 * T * (gate + 2 * on * d_ff * d)}


def tolerance(case):
    """About four times the measured error against ``exact``.  One token, and fp32 weights: sums of
    32-bit products (2e-7 to 4e-7).  16-bit and quantized weights in a batch: tokens as two bf16
    parts, 2^-16 of an element (5e-6 to 7e-6)."""
    if case["tokens"] == 1 or case["weights"] == "f32":
        return {"rel": 2e-6}
    return {"rel": 3e-5}


def _wide(s, name):
    """A weight matrix in 64 bits."""
    w = s[name]
    if s["weights"] == "i4":
        lo, hi = (w & 15).to(torch.int8), (w >> 4).to(torch.int8)
        w = torch.stack((lo, hi), dim=2).reshape(w.shape[0], -1)
        w = torch.where(w >= 8, w - 16, w)
    w = w.double()
    scale = s["scales"].get("lopa_b" if name == "gate" and s["r"] else name)
    return w if scale is None else w * scale.double()[:, None]


def exact(case, seed):
    s = prepare(case, seed)
    x = s["x"].double()
    form = s.get("form") or {}
    if case["r"]:
        z = x @ _wide(s, "lopa_a").t()
        if form:
            z = z / torch.sqrt((z * z).mean(1, keepdim=True) + RMS_EPS) * form["rms_gain"].double()
        h = z @ _wide(s, "gate").t()
        if form:
            h = h + x[:, form["g_idx"].long()] * form["g_sign"].double()
    else:
        h = x @ _wide(s, "gate").t()
    # the entry points take the threshold as a 32-bit number
    u = h - float(torch.tensor(s["t"], dtype=torch.float32))
    on = u > 0
    u = torch.where(on, u, torch.zeros_like(u))
    v = x @ _wide(s, "up").t()
    if case["full"]:
        u = u * torch.sigmoid(u)
        v = v * torch.sigmoid(v)
    return (u * v) @ _wide(s, "down")
