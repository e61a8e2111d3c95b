"""The work a user of the MoE-layer library has it do, as cases that can be timed and compared.

Three kinds of call, all through the package's public entry points:

  forward   moe_forward, the whole layer (route, permute, gate+up, down, combine) on resident weights: what a serving
            program calls once per layer and step.  `packed`: the weights are the copy that moe_pack_weights made at load
            time (the serving layout), or the row-major tensors themselves (the interchange layout).
  route     moe_route alone: a program that dispatches the tokens itself (expert parallelism) or only scores them.
  experts   moe_permute, moe_grouped_ffn and moe_combine on assignments that come from outside, as a program does that has
            its own router, or replays recorded routing.

Layer shapes are the repository's own (moe_inputs.PRESETS) or generic ones; a case is T tokens, model width d, expert width F,
E experts of which each token takes k, a gating rule, and `skew`: 0 for near-uniform routing, else the exponent of the power
law that the experts' popularity follows (as a logit bias for `forward` and `route`, as the distribution the assignments are
drawn from for `experts`).
"""
import math

import numpy as np
import torch

import moe_inputs as mi
import paper_2605_23911_amd as moe

DEV = "cuda:0"
BF16 = torch.bfloat16


def _preset(kind, preset, T, packed=True, skew=0.0, gating=None):
    s = mi.PRESETS[preset]
    return {"kind": kind, "T": T, "d": s.d, "F": s.F, "E": s.E, "k": s.k, "gating": s.gating if gating is None else gating,
            "packed": packed, "skew": skew}


def listed():
    named = {
        # A small layer on a handful of tokens: nothing but launches and latency.
        "tiny, 64 tokens": _preset("forward", "tiny", 64),
        # One user's decode step: two experts' weights are read for a single token.
        "mixtral, 1 token": _preset("forward", "mixtral", 1),
        # A decode batch of an odd size: every expert is hit by a few rows, the weights stream once.
        "mixtral, 47 tokens": _preset("forward", "mixtral", 47),
        # A large decode batch or a short prompt: bench.py's default workload.
        "mixtral, 512 tokens": _preset("forward", "mixtral", 512),
        # The same from the row-major tensors, as a program calls it that does not keep a packed copy.
        "mixtral, 512 tokens, row-major": _preset("forward", "mixtral", 512, packed=False),
        # Prefill: each expert holds about a thousand rows, the matrix cores bound the layer.
        "mixtral, 4096 tokens": _preset("forward", "mixtral", 4096),
        # Many mid-size experts, decode batch, weights renormalised over the chosen k.
        "qwen2moe, 100 tokens": _preset("forward", "qwen2moe", 100),
        # Prefill on many experts with popular and unpopular ones side by side.
        "qwen2moe, 4096 tokens, skew 1": _preset("forward", "qwen2moe", 4096, skew=1.0),
        # 256 experts of a few rows each: weight streaming over 22 GB.
        "dsv3, 512 tokens": _preset("forward", "dsv3", 512),
        # The largest: prefill on 256 experts, sigmoid gating.
        "dsv3, 4096 tokens, sigmoid": _preset("forward", "dsv3", 4096, gating=moe.GATE_SIGMOID_NORM),
        # The router alone on 256 experts.
        "router of 256, 1024 tokens": _preset("route", "dsv3", 1024),
        # Assignments from outside on a layer whose widths are no multiple of 128, an odd token count, uneven experts.
        "experts, ragged, 1001 tokens": {"kind": "experts", "T": 1001, "d": 2880, "F": 2880, "E": 32, "k": 4,
                                         "gating": moe.GATE_SOFTMAX, "packed": True, "skew": 1.0},
    }
    return [dict(c, name=n) for n, c in named.items()]


_MOST_FLOPS = 4096 * 6 * 8 * 7168 * 2048      # the largest listed case
_MOST_WEIGHTS = 6 * 256 * 7168 * 2048


def draw(rng):
    """One more case: any kind, a preset or a generic shape, T from 1 to 4096 over its logarithm, all gatings, both layouts."""
    kind = rng.choices(["forward", "route", "experts"], [7, 1, 2])[0]
    while True:
        if rng.random() < 0.6:
            s = mi.PRESETS[rng.choice(["mixtral", "qwen2moe", "dsv3", "mixtral22"])]
            d, F, E, k = s.d, s.F, s.E, s.k
        else:
            E = rng.choice([4, 7, 8, 16, 24, 32, 60, 64, 128, 160, 256])
            k = rng.randint(1, min(E, 8))
            d = 64 * round(math.exp(rng.uniform(math.log(8), math.log(112))))
            F = 64 * round(math.exp(rng.uniform(math.log(8), math.log(224))))
        T = round(math.exp(rng.uniform(0.0, math.log(4096.0))))
        if 6 * T * k * d * F <= _MOST_FLOPS and 6 * E * d * F <= _MOST_WEIGHTS:
            break
    return {"kind": kind, "T": T, "d": d, "F": F, "E": E, "k": k, "gating": rng.choice([0, 1, 2]),
            "packed": rng.random() < 0.8, "skew": rng.choice([0.0, 0.0, round(rng.uniform(0.3, 2.0), 2)])}


# ---- inputs -------------------------------------------------------------------------------------------------------------


def _normal(shape, std, seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1_000_003 + stream) * 4099)
    t = torch.empty(shape, dtype=BF16, device=DEV).normal_(generator=g)
    return t.mul_(std) if std != 1.0 else t


def _popularity(case, seed):
    """Shares of the experts: rank^-skew over a seeded ranking."""
    rank = np.random.default_rng([seed, 11]).permutation(case["E"]) + 1.0
    p = rank ** -float(case["skew"])
    return p / p.sum()


def _inputs(case, seed):
    """Activations ~ N(0, 1) and weights ~ N(0, 1/fan-in) in bf16, as the repository's own inputs."""
    T, d, F, E, k = (case[n] for n in ("T", "d", "F", "E", "k"))
    i = {"x": _normal((T, d), 1.0, seed, 0)}
    if case["kind"] == "experts":
        p = torch.from_numpy(_popularity(case, seed)).expand(T, E)
        g = torch.Generator().manual_seed(seed)
        i["topk_idx"] = torch.multinomial(p, k, generator=g).to(torch.int32).to(DEV)
        w = torch.rand((T, k), generator=g) + 0.1
        i["topk_w"] = (w / w.sum(1, keepdim=True)).to(DEV)
    else:
        i["wr"] = _normal((E, d), d ** -0.5, seed, 1)
        i["bias"] = torch.from_numpy(np.log(_popularity(case, seed)).astype(np.float32)).to(DEV) if case["skew"] else None
    if case["kind"] != "route":
        i["wg"] = _normal((E, F, d), d ** -0.5, seed, 2)
        i["wu"] = _normal((E, F, d), d ** -0.5, seed, 3)
        i["wd"] = _normal((E, d, F), F ** -0.5, seed, 4)
    return i


def prepare(case, seed):
    T, d, E, k = (case[n] for n in ("T", "d", "E", "k"))
    i = _inputs(case, seed)
    cfg = moe.MoEConfig.of(T, d, case["F"], E, k, case["gating"])
    s = {"kind": case["kind"], "cfg": cfg, "packed": None, **i}

    def buf(n, dtype=torch.uint8):
        return torch.empty(n, dtype=dtype, device=DEV)

    if case["kind"] == "route":
        s.update(topk_idx=buf((T, k), torch.int32), topk_w=buf((T, k), torch.float32), ws=buf(moe.route_workspace_size(cfg)))
        return s
    if case["packed"]:     # once at load time; the row-major tensors are not kept
        s["packed"] = buf(moe.packed_weights_size(cfg))
        moe.moe_pack_weights(cfg, s["wg"], s["wu"], s["wd"], s["packed"])
        s["wg"] = s["wu"] = s["wd"] = None
    s["y"] = buf((T, d), BF16)
    if case["kind"] == "forward":
        lay = moe.forward_workspace_layout(cfg)
        s["ws"] = buf(lay.total)
        s["topk_idx"] = s["ws"][lay.topk_idx: lay.topk_idx + 4 * T * k].view(torch.int32).view(T, k)
        s["topk_w"] = s["ws"][lay.topk_w: lay.topk_w + 4 * T * k].view(torch.float32).view(T, k)
        return s
    R = T * k
    s.update(counts=buf(E, torch.int32), offsets=buf(E + 1, torch.int32), row_of=buf(R, torch.int32), src_of=buf(R, torch.int32),
             x_perm=buf((R, d), BF16), h=buf((R, case["F"]), BF16), y_perm=buf((R, d), BF16),
             ws=buf(max(moe.permute_workspace_size(cfg), moe.ffn_workspace_size(cfg))))
    return s


def run(s):
    cfg = s["cfg"]
    if s["kind"] == "route":
        moe.moe_route(cfg, s["x"], s["wr"], s["bias"], s["topk_idx"], s["topk_w"], s["ws"])
        return {"topk_idx": s["topk_idx"], "topk_w": s["topk_w"]}
    if s["kind"] == "forward":
        moe.moe_forward(cfg, s["x"], s["wr"], s["bias"], s["wg"], s["wu"], s["wd"], s["y"], s["ws"], W_packed=s["packed"])
        return {"y": s["y"], "topk_idx": s["topk_idx"], "topk_w": s["topk_w"]}
    moe.moe_permute(cfg, s["x"], s["topk_idx"], s["counts"], s["offsets"], s["row_of"], s["src_of"], s["x_perm"], s["ws"])
    moe.moe_grouped_ffn(cfg, s["x_perm"], s["offsets"], s["wg"], s["wu"], s["wd"], s["h"], s["y_perm"], s["ws"], W_packed=s["packed"])
    moe.moe_combine(cfg, s["y_perm"], s["row_of"], s["topk_w"], s["y"])
    return {"y": s["y"], "h": s["h"], "y_perm": s["y_perm"], "offsets": s["offsets"], "row_of": s["row_of"], "src_of": s["src_of"]}


# ---- what it costs at least, how close results have to be, and what they are -------------------------------------------


def work(case):
    """Weights of the experts that are hit (in the mean, for uniform routing), activations in, results out."""
    T, d, F, E, k = (case[n] for n in ("T", "d", "F", "E", "k"))
    R = T * k
    router = {"bytes": 2 * E * d + 2 * T * d + 8 * R, "flops": 2 * T * E * d}
    if case["kind"] == "route":
        return router
    if case["skew"]:
        p = np.sort(_popularity(case, 0))
        hit = float((1 - (1 - np.minimum(1.0, p * k)) ** T).sum())
    else:
        hit = E * (1 - (1 - k / E) ** T)
    b = 6 * d * F * hit + 2 * T * d      # expert weights, y
    f = 6 * R * d * F
    if case["kind"] == "forward":
        return {"bytes": b + router["bytes"], "flops": f + router["flops"]}
    return {"bytes": b + 2 * T * d + 2 * R * d + 2 * R * F + 2 * R * d + 16 * R, "flops": f}   # x; x_perm, h, y_perm written


def tolerance(case):
    if case["kind"] == "route":
        # fp32 weights of an fp64 evaluation: one rounding
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    # bf16 results with two (forward) or three bf16 roundings on the way: about 3e-3 from exact()
    return {"rel": 1.2e-2, "max": 0.08, "differ": 0.0}


def exact(case, seed):
    """The layer in float64 by torch, expert by expert."""
    T, d, F, E, k = (case[n] for n in ("T", "d", "F", "E", "k"))
    i = _inputs(case, seed)
    x = i["x"].double()
    if case["kind"] == "experts":
        idx, w = i["topk_idx"].long(), i["topk_w"].double()
    else:
        z = x @ i["wr"].double().t()
        if i["bias"] is not None:
            z += i["bias"].double()
        top, idx = torch.topk(z, k, dim=1)
        if case["gating"] == 0:      # softmax over all experts
            w = torch.exp(top - torch.logsumexp(z, 1, keepdim=True))
        elif case["gating"] == 1:    # softmax over the chosen ones
            w = torch.softmax(top, 1)
        else:                        # sigmoid, normalised over the chosen ones
            w = torch.sigmoid(top)
            w = w / w.sum(1, keepdim=True)
        if case["kind"] == "route":
            return {"topk_idx": idx.int(), "topk_w": w}
    flat = idx.reshape(-1)
    src = torch.sort(flat, stable=True).indices       # expert-contiguous order
    off = torch.zeros(E + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(torch.bincount(flat, minlength=E), 0).cpu()
    full = case["kind"] == "experts"
    h = torch.empty((T * k, F), dtype=torch.float64, device=DEV) if full else None
    yp = torch.empty((T * k, d), dtype=torch.float64, device=DEV)
    for e in range(E):
        a, b = int(off[e]), int(off[e + 1])
        if a == b:
            continue
        xe = x[src[a:b] // k]
        he = torch.nn.functional.silu(xe @ i["wg"][e].double().t()) * (xe @ i["wu"][e].double().t())
        yp[a:b] = he @ i["wd"][e].double().t()
        if full:
            h[a:b] = he
    row = torch.empty_like(src)
    row[src] = torch.arange(T * k, device=DEV)
    y = torch.zeros((T, d), dtype=torch.float64, device=DEV)
    for j in range(k):
        y += w[:, j: j + 1] * yp[row.view(T, k)[:, j]]
    if full:
        return {"y": y, "h": h, "y_perm": yp, "offsets": off.int(), "row_of": row.int(), "src_of": src.int()}
    return {"y": y, "topk_idx": idx.int(), "topk_w": w}
