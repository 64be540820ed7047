"""The work that a user of the mixed-precision MoE layer has it do, as a list
of timed cases through the public binding: decode steps from one token to the
decode maximum, a decode stack on the residual stream, prefill from a small
ragged layer to the 8192-token maximum, the quantiser that builds expert
copies, and the expert predictor.

Shapes are the two models of the paper's Table 1 (Mixtral-8x7B: d_model 4096,
d_ff 14336, 8 experts, top-2; Phi-MoE: 4096, 6400, 16 experts, top-2) and the
small layers of the tests.  Hidden states are N(0, 1) and weights N(0, 0.02)
in fp16, as everywhere in this repository.
"""
from __future__ import annotations

import math

import torch

import paper_2411_01433_amd as P

TAG_FP16, TAG_INT4, TAG_INT2, TAG_MISS_INT4, TAG_MISS_INT2 = 0, 1, 2, 3, 4
TAG_INT8, TAG_MISS_INT8_INT2 = 5, 6
HIGH, LOW, SKIP = 0, 1, 2
RMS_EPS = 1e-5
W_STD = 0.02
DEV = "cuda"

MIXTRAL = {"d": 4096, "f": 14336, "E": 8, "K": 2}
PHI = {"d": 4096, "f": 6400, "E": 16, "K": 2}


def listed():
    return [
        # the expert predictor beside every decode step: the smallest call
        {"name": "predict_p4_t1", "kind": "predict", "d": 4096, "E": 8, "K": 2, "T": 1, "p": 4},
        # a small layer (the tests' tiny one): launches and latency only
        {"name": "tiny_decode_t4", "kind": "decode", "d": 256, "f": 512, "E": 8, "K": 2, "T": 4,
         "tags": "431"},
        # interactive serving, one sequence: cached fp16 experts, misses by the Eq. 2 rule
        {"name": "mixtral_decode_t1", "kind": "decode", **MIXTRAL, "T": 1, "tags": "miss4"},
        # the same for an int8 model (int8 high copies, int2 low copies, skips)
        {"name": "mixtral_int8_decode_t1", "kind": "decode", **MIXTRAL, "T": 1, "tags": "int8miss"},
        # a small batch whose tokens favour a few experts
        {"name": "mixtral_decode_t8_skew", "kind": "decode", **MIXTRAL, "T": 8, "tags": "431",
         "skew": True},
        # the largest decode batch a step takes
        {"name": "mixtral_decode_t64", "kind": "decode", **MIXTRAL, "T": 64, "tags": "431"},
        # a whole decode pass over stacked layers on the residual stream
        {"name": "phi_stack4_decode_t4", "kind": "stack", **PHI, "T": 4, "tags": "half",
         "layers": 4},
        # an odd, small layer in prefill: partial tiles everywhere
        {"name": "ragged_prefill_t200", "kind": "prefill", "d": 320, "f": 448, "E": 6, "K": 3,
         "T": 200, "tags": "431"},
        # a prompt of 512 tokens through one layer with the residual glue
        {"name": "mixtral_prefill_t512", "kind": "prefill", **MIXTRAL, "T": 512, "tags": "431",
         "residual": True},
        # a prompt of odd length on the model with more, smaller experts
        {"name": "phi_prefill_t1337", "kind": "prefill", **PHI, "T": 1337, "tags": "half"},
        # the largest prefill call: a long prompt or several batched
        {"name": "mixtral_prefill_t8192", "kind": "prefill", **MIXTRAL, "T": 8192, "tags": "431"},
        # building one matrix's int4 copy (an expert enters the low-precision cache)
        {"name": "quantize_int4_14336x4096", "kind": "quantize", "rows": 14336, "cols": 4096,
         "bits": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "prefill", "stack",
                       "quantize", "predict"])
    if kind == "quantize":
        rows = _log_int(rng, 64, 14336)
        return {"kind": kind, "rows": rows, "cols": 32 * _log_int(rng, 8, 448),
                "bits": rng.choice([8, 4, 2])}
    shape = rng.choice([MIXTRAL, PHI, None])
    if shape is None:
        E = rng.choice([4, 6, 8, 12, 16])
        shape = {"d": 64 * _log_int(rng, 4, 64), "f": 64 * _log_int(rng, 6, 128), "E": E,
                 "K": rng.choice([1, 2, 2, 3, 4])}
    if kind == "predict":
        return {"kind": kind, "d": shape["d"], "E": shape["E"], "K": shape["K"],
                "T": _log_int(rng, 1, 64), "p": rng.randint(1, 8)}
    tags = rng.choice(["fp16", "431", "half", "miss4", "int8miss"])
    if kind == "prefill":
        return {"kind": kind, **shape, "T": _log_int(rng, 16, 8192 * 2 // shape["K"] if
                                                     shape["K"] > 2 else 8192),
                "tags": tags, "skew": rng.random() < 0.25, "residual": rng.random() < 0.5}
    if kind == "stack":
        return {"kind": kind, **shape, "T": _log_int(rng, 1, 16), "tags": tags,
                "layers": rng.randint(2, 4)}
    return {"kind": kind, **shape, "T": _log_int(rng, 1, 64), "tags": tags,
            "skew": rng.random() < 0.25}


# ---- inputs ------------------------------------------------------------------

def _tags(recipe, E, seed):
    """Per-expert tags; the split over the experts is a seeded permutation."""
    g = torch.Generator().manual_seed(seed * 7919 + 17)
    perm = torch.randperm(E, generator=g).tolist()
    if recipe == "fp16":
        row = [TAG_FP16] * E
    elif recipe == "431":  # fp16 : int4 : int2 = 4 : 3 : 1
        n16, n4 = E * 4 // 8, E * 3 // 8
        row = [TAG_FP16] * n16 + [TAG_INT4] * n4 + [TAG_INT2] * (E - n16 - n4)
    elif recipe == "half":
        row = [TAG_FP16] * (E // 2) + [TAG_INT4] * (E - E // 2)
    elif recipe == "miss4":
        row = [TAG_FP16] * (E // 2) + [TAG_MISS_INT4] * (E - E // 2)
    else:  # int8miss
        row = [TAG_INT8] * (E // 2) + [TAG_MISS_INT8_INT2] * (E - E // 2)
    tags = [0] * E
    for i, e in enumerate(perm):
        tags[e] = row[i]
    return tags


def _thresholds(recipe):
    return {"miss4": (0.7, 1.0), "int8miss": (0.6, 0.9)}.get(recipe, (1.0, 1.0))


def _normal(g, shape, std):
    return torch.empty(shape, dtype=torch.float16, device=DEV).normal_(0.0, std, generator=g)


def _layer_weights(case, g):
    d, f, E = case["d"], case["f"], case["E"]
    wg = _normal(g, (E, d), W_STD)
    if case.get("skew"):
        wg *= 4
    w1 = [_normal(g, (f, d), W_STD) for _ in range(E)]
    w3 = [_normal(g, (f, d), W_STD) for _ in range(E)]
    w2 = [_normal(g, (d, f), W_STD) for _ in range(E)]
    return wg, w1, w3, w2


def _hidden(case, g):
    x = torch.empty((case["T"], case["d"]), device=DEV).normal_(generator=g)
    if case.get("skew"):  # tokens share a direction, so they favour the same experts
        x = (x + torch.empty((1, case["d"]), device=DEV).normal_(generator=g)) * math.sqrt(0.5)
    return x.half()


def _inputs(case, seed):
    """Everything that is made from the seed: weights, tags and activations."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    kind = case["kind"]
    if kind == "quantize":
        return {"w": _normal(g, (case["rows"], case["cols"]), W_STD)}
    if kind == "predict":
        gates = [_normal(g, (case["E"], case["d"]), W_STD) for _ in range(case["p"])]
        host = torch.Generator().manual_seed(seed)
        cached = torch.randint(0, 1 << case["E"], (case["p"],), generator=host)
        return {"gates": gates, "x": _hidden(case, g), "cached": cached.to(DEV)}
    n = case.get("layers", 1)
    layers = [_layer_weights(case, g) for _ in range(n)]
    tags = [_tags(case["tags"], case["E"], seed * 64 + i) for i in range(n)]
    s = {"layers": layers, "tags": tags, "x": _hidden(case, g)}
    if kind == "stack" or case.get("residual"):
        s["h0"] = torch.empty((case["T"], case["d"]), device=DEV).normal_(generator=g)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind = case["kind"]
    if kind == "quantize":
        r, c, b = case["rows"], case["cols"], case["bits"]
        s["codes"] = torch.empty((r, c * b // 8), dtype=torch.uint8, device=DEV)
        s["scales"] = torch.empty((r, c // 32), dtype=torch.float16, device=DEV)
        return s
    T, d, E, K = case["T"], case["d"], case["E"], case["K"]
    if kind == "predict":
        p = case["p"]
        s["pred"] = P.MoePredictor(d, E, K, T, s["gates"])
        s["idx"] = torch.empty((T, p, K), dtype=torch.int32, device=DEV)
        s["w"] = torch.empty((T, p, K), dtype=torch.float32, device=DEV)
        s["first"] = torch.empty(1, dtype=torch.int32, device=DEV)
        s["preload"] = torch.empty(1, dtype=torch.int64, device=DEV)
        return s
    t1, t2 = _thresholds(case["tags"])
    s["moe"] = []
    for (wg, w1, w3, w2), tags in zip(s["layers"], s["tags"]):
        L = P.MoeLayer(d, case["f"], E, K, T, wg, w1, w3, w2, t1=t1, t2=t2, rms_eps=RMS_EPS)
        for e, tag in enumerate(tags):
            if tag != TAG_FP16:
                L.set_expert_precision(e, tag)
        if s["moe"]:
            L.share_workspace(s["moe"][0])
        s["moe"].append(L)
    s["idx"] = torch.empty((T, K), dtype=torch.int32, device=DEV)
    s["w"] = torch.empty((T, K), dtype=torch.float32, device=DEV)
    s["prec"] = torch.empty((T, K), dtype=torch.int8, device=DEV)
    s["y"] = torch.empty((T, d), dtype=torch.float32, device=DEV)
    s["h"] = torch.empty((T, d), dtype=torch.float32, device=DEV)
    s["xn"] = torch.empty((T, d), dtype=torch.float16, device=DEV)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "quantize":
        P.quantize(s["w"], case["bits"], s["codes"], s["scales"])
        return {"codes": s["codes"], "scales": s["scales"]}
    if kind == "predict":
        s["pred"].predict(s["x"], s["cached"], s["idx"], s["first"], s["preload"], s["w"])
        return {"w": s["w"], "idx": s["idx"], "first": s["first"], "preload": s["preload"]}
    if kind == "stack":
        # the residual stream enters the stack (the embedding's output) and is updated in place
        s["h"].copy_(s["h0"])
        for L in s["moe"]:
            L.decode_step_prenorm(s["h"], s["xn"])
        return {"h": s["h"]}
    L = s["moe"][0]
    if kind == "decode":
        # the routing goes back to the cache manager beside the output
        L.decode_step(s["x"], s["y"], s["idx"], s["w"], s["prec"])
        return {"y": s["y"], "w": s["w"], "idx": s["idx"], "prec": s["prec"]}
    if case.get("residual"):
        s["h"].copy_(s["h0"])
        L.prefill_residual(s["x"], s["h"], s["xn"])
        return {"h": s["h"], "x": s["xn"]}
    L.prefill(s["x"], s["y"], s["idx"], s["w"], s["prec"])
    return {"y": s["y"], "w": s["w"], "idx": s["idx"], "prec": s["prec"]}


# ---- what a pass cannot do without -----------------------------------------------

_BYTES = {TAG_FP16: 2.0, TAG_INT4: 0.5625, TAG_INT2: 0.3125, TAG_INT8: 1.0625,
          TAG_MISS_INT4: (2.0 + 0.5625) / 2, TAG_MISS_INT8_INT2: (1.0625 + 0.3125) / 2}


def work(case):
    kind = case["kind"]
    if kind == "quantize":
        n = case["rows"] * case["cols"]
        return {"bytes": n * 2 + n * case["bits"] / 8 + n / 32 * 2, "flops": 4.0 * n}
    T, d, E, K = case["T"], case["d"], case["E"], case["K"]
    if kind == "predict":
        p = case["p"]
        return {"bytes": p * E * d * 2 + T * d * 2 + T * p * K * 8, "flops": 2.0 * T * p * E * d}
    f, n = case["f"], case.get("layers", 1)
    tags = _tags(case["tags"], E, 0)
    per = sum(_BYTES[t] for t in tags) / E
    # distinct experts that T independent tokens are expected to select
    experts = E * (1.0 - (1.0 - K / E) ** T) if K < E else E
    rows = T * d * (2 + 4)
    if kind == "stack" or case.get("residual"):
        rows = T * d * (4 + 4 + 2)
    return {"bytes": n * (experts * per * 3 * d * f + E * d * 2 + rows),
            "flops": n * (6.0 * T * K * d * f + 2.0 * T * E * d)}


def tolerance(case):
    kind = case["kind"]
    if kind == "quantize":
        return "exact"
    if kind == "predict":
        return {"rel": 1e-5, "differ": 0.005}
    # fp16 activations between the projections and fp16-rounded dequantised
    # weights on the matrix cores, 2^-11 each: against 64 bits a layer is
    # 2.1e-4 to 3.7e-4 off, a stack of four 5.4e-4
    return {"rel": 2e-3 if kind == "stack" else 1.5e-3, "differ": 0.005}


# ---- the same in 64 bits -----------------------------------------------------------

def _quantised(w, bits):
    """(codes as signed numbers, scales) of the group-32 symmetric quantiser:
    s = fp16(max|w| / qmax), q = clamp(rne(w / s), -qmax - 1, qmax)."""
    qmax = (1 << (bits - 1)) - 1
    g = w.double().reshape(w.shape[0], -1, 32)
    s = (g.abs().amax(-1) / qmax).half().double()
    q = torch.where(s[..., None] > 0, (g / s[..., None].clamp_min(1e-30)).round(), 0.0 * g)
    return q.clamp_(-qmax - 1, qmax), s


def _copy(w, bits):
    if bits == 16:
        return w.double()
    q, s = _quantised(w, bits)
    return (q * s[..., None]).reshape(w.shape)


def _top(x, wg, K):
    lg = x.double() @ wg.double().T
    v, idx = torch.sort(lg, dim=-1, descending=True, stable=True)
    return idx[:, :K], torch.softmax(v[:, :K], dim=-1)


def _layer(case, weights, tags, x):
    """(y, w) of Eq. 1 with the Eq. 2 rule for fp16 activations x."""
    wg, w1, w3, w2 = weights
    t1, t2 = _thresholds(case["tags"])
    idx, w = _top(x, wg, case["K"])
    score = torch.cumsum(w, -1) - w
    score[:, 0] = 0.0
    x64 = x.double()
    y = torch.zeros((x.shape[0], case["d"]), dtype=torch.float64, device=x.device)
    for e, tag in enumerate(tags):
        hi = 8 if tag in (TAG_INT8, TAG_MISS_INT8_INT2) else 16
        lo = 4 if tag in (TAG_INT4, TAG_MISS_INT4) else 2
        on = idx == e
        if tag in (TAG_FP16, TAG_INT8):
            parts = [(hi, on)]
        elif tag in (TAG_INT4, TAG_INT2):
            parts = [(lo, on)]
        else:
            top = torch.zeros_like(on)
            top[:, 0] = True
            high = top | (score <= t1)
            parts = [(hi, on & high), (lo, on & ~high & (score <= t2))]
        for bits, m in parts:
            tok, slot = torch.nonzero(m, as_tuple=True)
            if tok.numel() == 0:
                continue
            xt = x64[tok]
            a = xt @ _copy(w1[e], bits).T
            a = a * torch.sigmoid(a) * (xt @ _copy(w3[e], bits).T)
            y.index_add_(0, tok, w[tok, slot, None] * (a @ _copy(w2[e], bits).T))
    return y, w


def _norm(h):
    return (h / torch.sqrt((h * h).mean(-1, keepdim=True) + RMS_EPS)).half()


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "quantize":
        b = case["bits"]
        q, sc = _quantised(s["w"], b)
        u = (q + (1 << (b - 1))).to(torch.int64).reshape(case["rows"], -1, 8 // b)
        codes = (u << (b * torch.arange(8 // b, device=u.device))).sum(-1)
        return {"codes": codes.to(torch.uint8), "scales": sc}
    if kind == "predict":
        w = torch.stack([_top(s["x"], g, case["K"])[1] for g in s["gates"]], 1)
        return {"w": w, "idx": None, "first": None, "preload": None}
    if kind == "stack":
        h = s["h0"].double()
        for weights, tags in zip(s["layers"], s["tags"]):
            h = h + _layer(case, weights, tags, _norm(h))[0]
        return {"h": h}
    y, w = _layer(case, s["layers"][0], s["tags"][0], s["x"])
    if case.get("residual"):
        h = s["h0"].double() + y
        return {"h": h, "x": (h / torch.sqrt((h * h).mean(-1, keepdim=True) + RMS_EPS))}
    return {"y": y, "w": w, "idx": None, "prec": None}
