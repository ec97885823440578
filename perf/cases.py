"""The calls that the framework's users make, over the range of sizes that they make them at.

A case names one call (or one training step) through the public entry points of
``paper_2604_01622_amd``:

  kind "train"    ``forward(save=True)`` then ``backward``: a training step of the layer
  kind "forward"  the layer in inference (one sequence: single-sample decoding)
  kind "tc"       token choice, the policy that expert choice is compared with
  kind "route"    routing alone with the slot map and the token drop statistic
                  (api "noalloc": the entry point for callers that cannot allocate)

``api`` says how the program holds the layer: "layer" keeps a ``Layer`` (or
``TcLayer``) planned once, as a benchmark or a decoding loop does; "call" uses the
functions, which size and allocate what they need on every call.

Token groups (sequences) are written as text, "2048x8" or "700,333,1015"; ``t``
holds the mask ratio of each group for capacities c(t) = c_min + (c_max - c_min)
(1 - t), and ``c`` a fixed capacity factor.
"""
import math

import numpy as np
import torch

import paper_2604_01622_amd as ec


def _case(name, kind, groups, d, E, h, **more):
    case = {"kind": kind, "api": "call", "groups": groups, "d": d, "E": E, "h": h, "hs": 0,
            "dtype": "bf16", "c": 8.0, "t": "", "c_min": 4.0, "c_max": 12.0, "inv_tau": 1.0,
            "top_k": 0, "cf": 0.0, "w_std": 0.02}
    if name:
        case["name"] = name
    case.update(more)
    return case


_T8 = "0.71,0.05,0.93,0.38,0.52,0.17,0.86,0.29"


def listed():
    return [
        # the flagship: a training step of the 8B-A1B block on 8 masked sequences, the
        # capacity of each following its mask ratio (the benchmark's default workload)
        _case("train_8x2048_E64", "train", "2048x8", 2048, 64, 1024, api="layer", c=0.0, t=_T8),
        # the same block with its two shared experts, half the sequences
        _case("train_shared_4x2048", "train", "2048x4", 2048, 64, 1024, hs=2048, c=0.0,
              t="0.64,0.12,0.91,0.35"),
        # a micro-batch of one sequence (gradient accumulation, fine-tuning): short
        # expert buffers in every product of both directions
        _case("train_1x2048_E64", "train", "2048", 2048, 64, 1024, c=8.0),
        # packed documents of unequal length and widths that no tile divides
        _case("train_ragged_E40", "train", "1531,77,1999,640,1203", 1472, 40, 832, c=5.0,
              w_std=0.026, inv_tau=2.0),
        # inference over long sequences with finer experts and a sharper router
        _case("forward_4x4096_E128", "forward", "4096x4", 2048, 128, 768, c=8.0, inv_tau=2.0),
        # single-sample decoding: one step of the denoising loop, early (many masked
        # tokens chosen per expert) ...
        _case("decode_1x2048_E64", "forward", "2048", 2048, 64, 1024, api="layer", c=0.0, t="0.09"),
        # ... and the last step of a short sequence, where the weights are most of the work
        _case("decode_1x512_late", "forward", "512", 2048, 64, 1024, api="layer", c=0.0, t="1.0"),
        # the comparison policy, dropless top 8
        _case("tc_8x2048_top8", "tc", "2048x8", 2048, 64, 1024, api="layer", top_k=8, cf=0.0),
        # routing alone: which experts a batch would use, and how many tokens none chose
        _case("route_8x2048_E64", "route", "2048x8", 2048, 64, 1024, c=0.0, t=_T8),
        # routing one long document for a caller that cannot allocate
        _case("route_1x16384_E128", "route", "16384", 2048, 128, 768, api="noalloc", c=8.0),
        # fp32 storage: the smallest layer (a unit test, a toy model) ...
        _case("forward_f32_tiny", "forward", "128", 64, 8, 128, dtype="f32", c=2.0, w_std=0.125),
        # ... and a training step of a small model in full precision
        _case("train_f32_ragged", "train", "700,333,1015", 1024, 16, 512, dtype="f32", c=4.0,
              w_std=0.031),
    ]


def _lengths(case):
    out = []
    for part in case["groups"].split(","):
        n, _, times = part.partition("x")
        out += [int(n)] * (int(times) if times else 1)
    return out


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _width(rng, lo, hi):
    return max(1, round(_log(rng, lo, hi) / 64)) * 64


def draw(rng):
    """One more case: another kind, other group lengths (odd ones among them), widths,
    expert counts, capacities and temperatures."""
    most = {c["name"]: c for c in listed()}
    while True:
        what = rng.choice(["train", "train", "train", "forward", "decode", "decode", "tc", "route",
                           "route", "f32", "f32"])
        E = rng.choice([8, 16, 24, 32, 40, 64, 64, 96, 128])
        inv_tau = rng.choice([0.5, 1.0, 1.0, 2.0])
        api = rng.choice(["layer", "call"])
        c = round(rng.uniform(2.0, min(12.0, E / 2)), 2)
        if what == "f32":
            kind = rng.choice(["train", "forward"])
            d, h, n = _width(rng, 64, 1024), _width(rng, 64, 512), rng.randint(1, 3)
            E = rng.choice([4, 8, 16, 17, 32])
            c = round(rng.uniform(1.0, min(4.0, E / 2)), 2)
            lens, limit = [int(_log(rng, 60, 1024)) for _ in range(n)], most["train_f32_ragged"]
        else:
            kind = "forward" if what == "decode" else what
            d, h = _width(rng, 512, 2560), _width(rng, 256, 1536)
            lens, limit = [int(_log(rng, 200, 4096)) for _ in range(rng.randint(1, 8))], \
                most["train_8x2048_E64"]
            if rng.random() < 0.4:
                lens = [rng.choice([512, 1024, 2048, 4096])] * rng.randint(1, 8)
            if what == "decode":
                lens = [int(_log(rng, 256, 4096))]
            if what == "route":
                limit = most["route_1x16384_E128"]
                api = rng.choice(["call", "noalloc"])
                if rng.random() < 0.3:
                    lens = [int(_log(rng, 4096, 16384))]
        case = _case("", kind, ",".join(map(str, lens)), d, E, h, inv_tau=inv_tau, api=api, c=c,
                     dtype="f32" if what == "f32" else "bf16", w_std=round(1.0 / math.sqrt(d), 4))
        if what in ("train", "forward", "decode") and rng.random() < 0.6:
            case["c"], case["c_max"] = 0.0, round(min(12.0, E / 2), 1)
            case["c_min"] = min(4.0, case["c_max"] / 2)
            case["t"] = ",".join("%.2f" % rng.random() for _ in lens)
        if what in ("train", "forward") and rng.random() < 0.25:
            case["hs"] = _width(rng, 256, 2048)
        if what == "tc":
            case["top_k"] = rng.choice([1, 2, 4, 8])
            case["cf"] = rng.choice([0.0, 1.0, 1.25])
        w, top = work(case), work(limit)
        if w["flops"] <= top["flops"] and w["bytes"] <= top["bytes"]:
            return case


def _capacity(case):
    """Tokens that each expert takes from each group, in plain arithmetic."""
    lens = _lengths(case)
    if case["kind"] == "tc":
        cf, k, E = case["cf"], case["top_k"], case["E"]
        return [n if cf <= 0 else min(n, math.ceil(cf * k * n / E - 1e-9)) for n in lens]
    if case["t"]:
        ts = [float(x) for x in case["t"].split(",")]
        lo, hi = case["c_min"], case["c_max"]
        cs = [min(hi, max(lo, lo + (hi - lo) * (1.0 - t))) for t in ts]
    else:
        cs = [case["c"]] * len(lens)
    return [int(min(n, max(0.0, np.rint(n * c / case["E"])))) for n, c in zip(lens, cs)]


def _inputs(case, seed):
    """X, Wg, W1, W3, W2, dY and the shared experts' weights, from the seed alone."""
    N, d, E, h, hs = sum(_lengths(case)), case["d"], case["E"], case["h"], case["hs"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device="cuda")

    def normal(i, shape, std):
        gen.manual_seed(seed * 16 + i)
        return (torch.randn(shape, generator=gen, device="cuda") * std).to(dt)

    w = case["w_std"]
    v = {"X": normal(0, (N, d), 1.0), "Wg": normal(1, (E, d), w)}
    if case["kind"] != "route":
        v["W1"], v["W3"] = normal(2, (E, h, d), w), normal(3, (E, h, d), w)
        v["W2"] = normal(4, (E, d, h), w)
    if case["kind"] == "train":
        v["dY"] = normal(5, (N, d), 1.0)
    v["shared"] = None
    if hs:
        v["shared"] = (normal(6, (hs, d), w), normal(7, (hs, d), w), normal(8, (d, hs), w))
    return v


def prepare(case, seed):
    lens = _lengths(case)
    st = _inputs(case, seed)
    st["case"] = case
    st["off"] = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    if case["kind"] == "tc":
        st["cap"] = ec.tc_capacity(lens, case["E"], case["top_k"], case["cf"])
    elif case["t"]:
        st["cap"] = ec.capacity(lens, case["E"], t=[float(x) for x in case["t"].split(",")],
                                c_min=case["c_min"], c_max=case["c_max"])
    else:
        st["cap"] = ec.capacity(lens, case["E"], c=case["c"])
    if case["api"] == "layer":
        weights = (st["X"], st["Wg"], st["W1"], st["W3"], st["W2"], st["off"], st["cap"])
        if case["kind"] == "tc":
            st["layer"] = ec.TcLayer(*weights, case["top_k"], case["inv_tau"], shared=st["shared"])
        else:
            st["layer"] = ec.Layer(*weights, case["inv_tau"], training=case["kind"] == "train",
                                   shared=st["shared"])
    return st


_GRADS = ("dX", "dWg", "dW1", "dW3", "dW2", "dWs1", "dWs3", "dWs2")


def run(st):
    case = st["case"]
    layer, tau, shared = st.get("layer"), case["inv_tau"], st["shared"]
    if case["kind"] == "route":
        call = ec.route_noalloc if case["api"] == "noalloc" else ec.route
        S, sel, gate, slot = call(st["X"], st["Wg"], st["off"], st["cap"], tau, d_ff=case["h"])
        count, dropped = ec.token_coverage(slot, st["off"], st["cap"], case["d"], case["h"])
        return {"S": S, "sel": sel, "gate": gate, "slot": slot, "count": count, "dropped": dropped}
    args = (st["X"], st["Wg"], st["W1"], st["W3"], st["W2"])
    if case["kind"] == "tc":
        if layer is not None:
            return {"Y": layer.forward(), "rows": layer.rows}
        Y, rows = ec.tc_forward(*args, st["off"], st["cap"], case["top_k"], tau, shared=shared)
        return {"Y": Y, "rows": rows}
    if case["kind"] == "forward":
        if layer is not None:
            return {"Y": layer.forward()}
        return {"Y": ec.forward(*args, st["off"], st["cap"], tau, shared=shared)}
    if layer is not None:
        Y = layer.forward()
        grads = tuple(layer.backward(st["dY"])) + tuple(layer.dshared or ())
    else:
        Y, saved = ec.forward(*args, st["off"], st["cap"], tau, save=True, shared=shared)
        grads = ec.backward(*args, st["dY"], saved, st["off"], st["cap"], tau, shared=shared)
    return {"Y": Y, **dict(zip(_GRADS, grads))}


def _pairs(case):
    """Token-expert pairs that are computed (token choice: the expected number kept)."""
    N, cap = sum(_lengths(case)), sum(_capacity(case))
    if case["kind"] == "tc":
        return min(case["top_k"] * N, case["E"] * cap)
    return case["E"] * cap


def work(case):
    N, d, E, h, hs = sum(_lengths(case)), case["d"], case["E"], case["h"], case["hs"]
    size = 2 if case["dtype"] == "bf16" else 4
    pairs = _pairs(case)
    router = 2 * N * d * E
    if case["kind"] == "route":
        # X and Wg in; S, slot map, selection, gates and counts out (the statistic
        # reads the slot map back)
        return {"bytes": (N + E) * d * size + 3 * N * E * 4 + 8 * pairs + 4 * N, "flops": router}
    weights = (E * d + 3 * E * d * h + 3 * d * hs) * size
    flops = 6 * d * (h * pairs + hs * N) + router
    if case["kind"] != "train":
        return {"bytes": 2 * N * d * size + weights, "flops": flops}
    # X, dY and the weights in; Y, dX and the weight gradients out (dWg in fp32)
    return {"bytes": 4 * N * d * size + 2 * weights + E * d * (4 - size), "flops": 3 * flops}


def tolerance(case):
    # fp32: sums of up to a few thousand terms.  Measured against 64 bits: scores
    # 2.5e-7, outputs and gradients up to 1.1e-6.
    # bf16: every stored activation and result is rounded once to 8 bits; measured
    # against 64 bits: 2.4e-3 to 3.6e-3 for outputs and gradients.
    # "differ" covers a pair of scores at an expert's threshold that another order of
    # the router's sums exchanges (it moves the places behind it in that expert's list),
    # and "max" the output rows of such a pair, where one of a token's experts is another.
    if case["kind"] == "route":
        return {"rel": 1e-6, "max": 2e-5, "differ": 2e-3}
    if case["dtype"] == "f32":
        return {"rel": 4.4e-6, "max": 1e-4, "differ": 2e-3}
    return {"rel": 1.2e-2, "max": 0.9, "differ": 2e-3}


# ---- the same calls in 64 bits, in plain torch --------------------------------


def _scores64(case, v):
    logits = v["X"].double() @ v["Wg"].double().t() * case["inv_tau"]
    return torch.softmax(logits, dim=1)


def _expert_choice64(case, S):
    """Tokens of each expert [E, K], ascending inside a group (ties: the lower token)."""
    off = np.concatenate([[0], np.cumsum(_lengths(case))])
    parts = []
    for g, k in enumerate(_capacity(case)):
        seg = S[off[g]:off[g + 1]]
        order = torch.sort(seg, dim=0, descending=True, stable=True).indices[:k]
        parts.append(torch.sort(order, dim=0).values.t() + int(off[g]))
    return torch.cat(parts, dim=1)


def _token_choice64(case, S):
    """Weights [N, E] of the kept pairs, 0 elsewhere."""
    k = case["top_k"]
    best = torch.sort(S, dim=1, descending=True, stable=True).indices[:, :k]
    chosen = torch.zeros_like(S).scatter_(1, best, 1.0)
    G = S * chosen
    G = G / G.sum(1, keepdim=True)
    off = np.concatenate([[0], np.cumsum(_lengths(case))])
    for g, cap in enumerate(_capacity(case)):
        seg = chosen[off[g]:off[g + 1]]
        G[off[g]:off[g + 1]] *= (torch.cumsum(seg, 0) <= cap) * seg
    return G


def _swiglu64(x, w1, w3):
    h1, h3 = x @ w1.t(), x @ w3.t()
    s = torch.sigmoid(h1)
    return h1, h3, s, h1 * s * h3


def _swiglu_back64(x, dy, w1, w3, w2, g):
    """Gradients of sum(dy * g * ffn(x)) for one expert: dx, dw1, dw3, dw2, <dy, ffn(x)>."""
    h1, h3, s, a = _swiglu64(x, w1, w3)
    raw = dy @ w2
    da = raw * g
    dh3 = da * h1 * s
    dh1 = da * h3 * s * (1 + h1 * (1 - s))
    return dh1 @ w1 + dh3 @ w3, dh1.t() @ x, dh3.t() @ x, (dy * g).t() @ a, (raw * a).sum(1)


def exact(case, seed):
    v = _inputs(case, seed)
    S = _scores64(case, v)
    if case["kind"] == "route":
        # the places in the lists are whole numbers, and the gates stand in their order
        return {"S": S, "sel": None, "gate": None, "slot": None, "count": None, "dropped": None}
    X, E = v["X"].double(), case["E"]
    Y = torch.zeros_like(X)
    if case["kind"] == "tc":
        G = _token_choice64(case, S)
        tokens = [torch.nonzero(G[:, j])[:, 0] for j in range(E)]
    else:
        G, tokens = S, _expert_choice64(case, S)
    for j in range(E):
        i = tokens[j]
        a = _swiglu64(X[i], v["W1"][j].double(), v["W3"][j].double())[3]
        Y[i] += G[i, j, None] * (a @ v["W2"][j].double().t())
    if v["shared"] is not None:
        w1, w3, w2 = (w.double() for w in v["shared"])
        Y += _swiglu64(X, w1, w3)[3] @ w2.t()
    if case["kind"] == "tc":
        return {"Y": Y, "rows": None}
    if case["kind"] == "forward":
        return {"Y": Y}
    dY, dX, dS = v["dY"].double(), torch.zeros_like(X), torch.zeros_like(S)
    dW1, dW3 = (torch.empty(v["W1"].shape, dtype=torch.float64, device="cuda") for _ in range(2))
    dW2 = torch.empty(v["W2"].shape, dtype=torch.float64, device="cuda")
    for j in range(E):
        i = tokens[j]
        dx, dW1[j], dW3[j], dW2[j], dS[i, j] = _swiglu_back64(
            X[i], dY[i], v["W1"][j].double(), v["W3"][j].double(), v["W2"][j].double(),
            S[i, j, None])
        dX[i] += dx
    dZ = S * (dS - (S * dS).sum(1, keepdim=True)) * case["inv_tau"]
    dX += dZ @ v["Wg"].double()
    out = {"Y": Y, "dX": dX, "dWg": dZ.t() @ X, "dW1": dW1, "dW3": dW3, "dW2": dW2}
    if v["shared"] is not None:
        dx, out["dWs1"], out["dWs3"], out["dWs2"], _ = _swiglu_back64(X, dY, w1, w3, w2, 1.0)
        dX += dx
    return out
