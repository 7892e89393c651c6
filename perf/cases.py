"""Workloads of the MoE expert layer, for timing and for comparing two builds of the library.

A case is one of four kinds, each a call sequence a user's program makes through the package:

  step     LayerState.forward() + backward(): a training step of one MoE layer (routing, permute, expert MLP, combine,
           and all gradients), in bf16, all-fp32, blockwise fp8 or MXFP8
  forward  LayerState.forward(): inference, from a handful of decoding tokens to a prefill
  gate     moe_gate_gemm: the router's projection, fp32 logits from bf16 activations
  router   moe_route_topk(_grouped), moe_aux_loss and moe_route_topk_bwd on given logits: the router of a training step

Inputs are drawn here, on the device, from the seed alone.  `exact` states the same results in 64-bit torch
arithmetic without calling the library.
"""
import math

import numpy as np
import torch

from paper_2603_07685_amd import binding as B
from paper_2603_07685_amd import layer as L
from paper_2603_07685_amd import workloads as wl

_STEP = dict(kind="step", recipe="bf16", T=0, h=0, f=0, E=0, k=0, E_router=0, score="softmax", norm_topk=False,
             n_group=1, topk_group=1, scale=1.0, bias=False, load="router", shared_f=0, eq2=False, gather=False,
             wgrad_f32=False)
_ROUTER = dict(kind="router", T=0, E=0, k=0, score="sigmoid", norm_topk=True, n_group=1, topk_group=1, scale=1.0, bias=False)


def _step(name, **kw):
    return dict(_STEP, name=name, **kw)


def listed():
    return [
        # the smallest layer of the repository's own configurations: nothing but launches and latency
        _step("step_tiny_bf16", T=256, h=128, f=256, E=8, k=2, E_router=8),
        # a small research model's layer
        _step("step_mid_bf16", T=2048, h=1024, f=512, E=8, k=2, E_router=8),
        # the same layer in fp32 end to end, the type of numerical studies
        _step("step_mid_fp32", recipe="fp32", T=2048, h=1024, f=512, E=8, k=2, E_router=8),
        # a small layer in the blockwise one-byte recipe, with a shared expert
        _step("step_small_fp8", recipe="fp8", T=1024, h=512, f=256, E=8, k=4, E_router=32, score="sigmoid",
              norm_topk=True, load="cv", shared_f=256),
        # sizes off every power of two, MXFP8
        _step("step_odd_mxfp8", recipe="mxfp8", T=3968, h=1920, f=896, E=13, k=3, E_router=13),
        # sizes off every power of two, bf16: the group-limited router with bias, a shared expert, fp32 main gradients
        _step("step_odd_grouped_bf16", T=1999, h=2880, f=1472, E=24, k=4, E_router=24, score="sigmoid", norm_topk=True,
              n_group=4, topk_group=2, scale=2.5, bias=True, shared_f=1472, wgrad_f32=True),
        # decoding: a few tokens on each expert of a Qwen3-235B-style share, bound by reading the weights
        dict(_step("forward_decode_bf16", T=64, h=4096, f=1536, E=16, k=8, E_router=128, load="cv"), kind="forward"),
        # Qwen3-235B-style share, strongly unequal experts, weights before fc2 and the permute inside the GEMMs
        _step("step_qwen3_zipf_bf16", T=16384, h=4096, f=1536, E=16, k=8, E_router=128, load="zipf", eq2=True,
              gather=True),
        # DeepSeek-V3-style share: the largest, and the one the repository's benchmark times
        _step("step_dsv3_bf16", T=16384, h=7168, f=2048, E=32, k=8, E_router=256, score="sigmoid", norm_topk=True,
              load="cv", shared_f=2048),
        _step("step_dsv3_mxfp8", recipe="mxfp8", T=16384, h=7168, f=2048, E=32, k=8, E_router=256, score="sigmoid",
              norm_topk=True, load="cv", shared_f=2048),
        # the router's projection and the router itself at the DeepSeek-V3 sizes
        dict(name="gate_dsv3", kind="gate", T=16384, E=256, h=7168),
        dict(_ROUTER, name="router_dsv3_grouped", T=16384, E=256, k=8, n_group=8, topk_group=4, scale=2.5, bias=True),
    ]


# --- drawn cases ----------------------------------------------------------------------------------------------------
def _log(rng, lo, hi, step=1):
    """A multiple of `step` between lo and hi, uniform over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi // step * step, max(-(-lo // step) * step, int(round(v / step)) * step))


def _score(rng):
    return dict(score=rng.choice(("softmax", "sigmoid")), norm_topk=rng.random() < 0.5)


def draw(rng):
    kind = rng.choice(("step", "step", "step", "step", "forward", "forward", "gate", "router"))
    if kind == "gate":
        return dict(kind="gate", T=_log(rng, 16, 16384), E=_log(rng, 8, 256, 8), h=_log(rng, 128, 7168, 64))
    if kind == "router":
        c = dict(_ROUTER, T=_log(rng, 16, 16384), **_score(rng))
        if rng.random() < 0.5:
            c["n_group"] = rng.choice((2, 4, 8))
            c["topk_group"] = c["n_group"] // 2
            c["E"] = c["n_group"] * _log(rng, 4, 32)
            c["k"] = c["topk_group"] * rng.choice((1, 2))
            c.update(scale=2.5, bias=True)
        else:
            c["E"] = _log(rng, 8, 256)
            c["k"] = min(rng.choice((1, 2, 4, 6, 8)), c["E"])
        c["norm_topk"] = c["norm_topk"] and c["k"] > 1     # (one weight over itself: nothing to normalise)
        return c
    while True:
        c = dict(_STEP, kind=kind, recipe=rng.choice(("bf16", "bf16", "bf16", "mxfp8", "fp8", "fp32")), **_score(rng))
        q = 128 if c["recipe"] in ("mxfp8", "fp8") else 64
        c["T"] = _log(rng, 128, 16384, 128) if q == 128 else _log(rng, 16, 16384)
        c["h"], c["f"] = _log(rng, 128, 7168, q), _log(rng, 128, 4096, q)
        c["E"] = _log(rng, 4, 64)
        c["k"] = min(rng.choice((1, 2, 4, 6, 8)), c["E"])
        c["norm_topk"] = c["norm_topk"] and c["k"] > 1
        c["load"] = rng.choice(("router", "cv", "zipf"))
        c["E_router"] = c["E"] if c["load"] == "router" else c["E"] * rng.choice((1, 2, 8))
        if rng.random() < 0.3:
            c["shared_f"] = c["f"]
        if c["recipe"] == "bf16":
            c["gather"] = rng.random() < 0.3
            c["wgrad_f32"] = rng.random() < 0.3
        if c["recipe"] != "fp32":
            c["eq2"] = rng.random() < 0.3
        big = listed()[2 if c["recipe"] == "fp32" else 8]
        if _flops(c) <= _flops(big) and c["E"] * c["h"] * c["f"] <= big["E"] * big["h"] * big["f"] and \
                c["T"] * c["k"] * max(c["h"], 2 * c["f"]) <= big["T"] * big["k"] * big["h"]:
            return c


# --- inputs ---------------------------------------------------------------------------------------------------------
def _inputs(case, seed):
    """Device tensors of a case: unit-variance activations and gradients, N(0, 0.02^2) weights, unit-variance logits."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def n(*shape, std=1.0, dt=torch.bfloat16):
        return torch.empty(shape, dtype=dt, device="cuda").normal_(0.0, std, generator=g)

    f32 = torch.float32
    T, h = case["T"], case.get("h", 0)
    if case["kind"] == "gate":
        return {"X": n(T, h), "Wr": n(case["E"], h, std=0.02)}
    E, k = case["E"], case["k"]
    d = {"logits": n(T, case.get("E_router", E), dt=f32)}
    if case["bias"]:
        d["bias"] = n(case.get("E_router", E), std=0.1, dt=f32)
    if case["kind"] == "router":
        d["dprob"] = n(T, k, dt=f32)
        return d
    f, sf = case["f"], case["shared_f"]
    d["X"], d["W1"], d["W2"] = n(T, h), n(E, 2 * f, h, std=0.02), n(E, h, f, std=0.02)
    if case["kind"] == "step":
        d["dY"] = n(T, h)
    if sf:
        d["Ws1"], d["Ws2"] = n(2 * sf, h, std=0.02), n(h, sf, std=0.02)
    if case["load"] != "router":
        # rows that the local experts receive, from this GPU's tokens and from other ranks': shares that scatter by
        # 30 % around the mean, or that fall as rank^-1.2 in a random order of the experts
        if case["load"] == "cv":
            w = (1.0 + 0.3 * n(E, dt=f32)).clamp(min=0.05)
        else:
            w = (1.0 + torch.randperm(E, generator=g, device="cuda")).to(f32) ** -1.2
        d["idx"] = torch.multinomial(w, T * k, replacement=True, generator=g).to(torch.int32).view(T, k)
    return d


_SCORE = {"softmax": wl.SOFTMAX, "sigmoid": wl.SIGMOID}


def prepare(case, seed):
    d = _inputs(case, seed)
    T, E = case["T"], case["E"]
    if case["kind"] == "gate":
        return {"case": case, "ctx": B.Context(T, 1, E, case["h"], E), **d,
                "logits": torch.empty((T, E), dtype=torch.float32, device="cuda")}
    if case["kind"] == "router":
        k, dev = case["k"], "cuda"
        return {"case": case, "ctx": B.Context(T, k, E, 64, 64), "bias": None, **d,
                "idx": torch.empty((T, k), dtype=torch.int32, device=dev),
                "prob": torch.empty((T, k), dtype=torch.float32, device=dev),
                "counts": torch.empty(E, dtype=torch.int32, device=dev),
                "loss": torch.empty(1, dtype=torch.float32, device=dev),
                "dlogits": torch.empty((T, E), dtype=torch.float32, device=dev)}
    one_byte = case["recipe"] in ("fp8", "mxfp8")
    cfg = wl.MoEConfig("perf", T=T, h=case["h"], f=case["f"], E=E, k=case["k"], E_router=case["E_router"],
                       score=_SCORE[case["score"]], norm_topk=case["norm_topk"],
                       load="router" if case["load"] == "router" else "uniform", shared_f=case["shared_f"],
                       fp8=case["recipe"] == "fp8", mx=case["recipe"] == "mxfp8", align=128 if one_byte else 1, seed=seed,
                       n_group=case["n_group"], topk_group=case["topk_group"], route_scale=case["scale"],
                       bias_std=0.1 if case["bias"] else 0.0)
    f32 = case["recipe"] == "fp32"
    hin = None
    if f32:
        hin = {n: d[n].float().cpu().numpy() for n in ("X", "W1", "W2", "Ws1", "Ws2", "logits") if n in d}
        hin["dY"] = d["dY"].float().cpu().numpy() if "dY" in d else np.zeros((T, case["h"]), np.float32)
    st = L.LayerState(cfg, hin, wgrad_f32=case["wgrad_f32"], eq2=case["eq2"], f32=f32, gather=case["gather"])
    for name, t in d.items():
        to = {"bias": "expert_bias", "idx": "forced_idx"}.get(name, name)
        getattr(st, to).copy_(t)
    return {"case": case, "layer": st}


# --- one pass -------------------------------------------------------------------------------------------------------
def run(s):
    c = s["case"]
    if c["kind"] == "gate":
        B.moe_gate_gemm(s["ctx"], s["X"], s["Wr"], c["T"], c["E"], c["h"], s["logits"])
        return {"logits": s["logits"]}
    if c["kind"] == "router":
        T, E, k, fn = c["T"], c["E"], c["k"], _SCORE[c["score"]]
        if c["n_group"] > 1 or c["bias"]:
            B.moe_route_topk_grouped(s["ctx"], s["logits"], s["bias"], T, E, k, c["n_group"], c["topk_group"], fn,
                                     c["norm_topk"], c["scale"], s["idx"], s["prob"], s["counts"])
        else:
            B.moe_route_topk(s["ctx"], s["logits"], T, E, k, fn, c["norm_topk"], c["scale"], s["idx"], s["prob"], s["counts"])
        B.moe_route_topk_bwd(s["ctx"], s["logits"], s["idx"], s["dprob"], T, E, k, fn, c["norm_topk"], c["scale"], s["dlogits"])
        B.moe_aux_loss(s["ctx"], s["logits"], s["counts"], T, E, k, fn, 0.01, 1.0, 1, s["loss"], s["dlogits"])
        return {n: s[n] for n in ("idx", "prob", "counts", "loss", "dlogits")}
    st = s["layer"]
    st.forward()
    out = {"idx": st.topk_idx, "prob": st.topk_prob, "row_of": st.row_of, "offsets": st.offsets, "Y": st.Y}
    if c["kind"] == "step":
        st.backward()
        out.update(dX=st.dX, dprob=st.dprob, dW1=st.dW1, dW2=st.dW2)
        if c["shared_f"]:
            out.update(dWs1=st.dWs1, dWs2=st.dWs2)
    return out


# --- what a pass cannot do without ----------------------------------------------------------------------------------
def _flops(c):
    passes = 3 if c["kind"] == "step" else 1
    return 6.0 * passes * c["h"] * (c["T"] * c["k"] * c["f"] + c["T"] * c["shared_f"])


def work(case):
    T, E = case["T"], case["E"]
    if case["kind"] == "gate":
        return {"bytes": 2.0 * (T + E) * case["h"] + 4.0 * T * E, "flops": 2.0 * T * E * case["h"]}
    if case["kind"] == "router":
        # logits in; indices, weights, their gradients; gradient of the logits out
        return {"bytes": 8.0 * T * E + 12.0 * T * case["k"] + 8.0 * E, "flops": 10.0 * T * E}
    h, f, k, sf = case["h"], case["f"], case["k"], case["shared_f"]
    es = 4 if case["recipe"] == "fp32" else 2                  # activations, gradients, weights as the caller holds them
    wes = 4 if case["wgrad_f32"] else es
    weights = 3.0 * h * (E * f + sf)
    b = 2.0 * T * h * es + weights * es + 4.0 * T * case["E_router"] + 12.0 * T * k
    if case["kind"] == "step":
        b += 2.0 * T * h * es + weights * wes + 4.0 * T * k
    return {"bytes": b, "flops": _flops(case)}


def tolerance(case):
    if case["kind"] == "gate":
        return {"rel": 1e-5}
    if case["kind"] == "router":
        return {"rel": 1e-5}
    return {"bf16": {"rel": 1e-2}, "fp32": {"rel": 1e-5}, "fp8": {"rel": 2e-2}, "mxfp8": {"rel": 2e-2}}[case["recipe"]]


# --- the same in 64 bits --------------------------------------------------------------------------------------------
def _scores(logits, score):
    x = logits.double()
    return torch.softmax(x, 1) if score == "softmax" else torch.sigmoid(x)


def _best(v, n):
    """Indices of the n largest of each row, largest first, ties to the lower index."""
    return torch.sort(v, dim=1, descending=True, stable=True)[1][:, :n]


def _route(c, logits, bias):
    """Selected experts and their weights.  The group-limited router decides on scores rounded to fp32, with fp32 sums."""
    k, s = c["k"], _scores(logits, c["score"])
    if c["n_group"] > 1 or c["bias"]:
        v = s.float()
        s = v.double()
        if bias is not None:
            v = v + bias
        T, E = v.shape
        if c["n_group"] > 1:
            m = k // c["topk_group"]
            top = torch.sort(v.view(T, c["n_group"], -1), dim=2, descending=True)[0][:, :, :m]
            gsum = top[:, :, 0]
            for r in range(1, m):
                gsum = gsum + top[:, :, r]
            keep = torch.zeros((T, c["n_group"]), dtype=torch.bool, device=v.device)
            keep.scatter_(1, _best(gsum, c["topk_group"]), True)
            v = v.masked_fill(~keep.repeat_interleave(E // c["n_group"], 1), -math.inf)
        idx = _best(v, k)
    else:
        idx = _best(logits, k)
    p = s.gather(1, idx)
    w = p / p.sum(1, keepdim=True) if c["norm_topk"] else p
    return idx, w * c["scale"]


def _exact_router(c, d):
    idx, prob = _route(c, d["logits"], d.get("bias"))
    T, E, k = c["T"], c["E"], c["k"]
    x = d["logits"].double().requires_grad_()
    with torch.enable_grad():
        s = torch.softmax(x, 1) if c["score"] == "softmax" else torch.sigmoid(x)
        q = s.gather(1, idx)
        w = (q / q.sum(1, keepdim=True) if c["norm_topk"] else q) * c["scale"]
        p = s if c["score"] == "softmax" else s / s.sum(1, keepdim=True)
        counts = torch.bincount(idx.flatten(), minlength=E)
        loss = 0.01 * E * ((counts.double() / (T * k)) * p.mean(0)).sum()
        ((w * d["dprob"].double()).sum() + loss).backward()
    return {"idx": idx.to(torch.int32), "prob": prob, "counts": counts.to(torch.int32), "loss": loss.detach().view(1),
            "dlogits": x.grad}


def _mlp(x, w1, w2, p, dy):
    """Rows x through one expert: output and, with the rows' gradient dy of p * output, (dx, dp, dw1, dw2)."""
    x, w1, w2 = x.double(), w1.double(), w2.double()
    g, u = (x @ w1.t()).chunk(2, 1)
    s = torch.sigmoid(g)
    a = g * s * u
    o = a @ w2.t()
    if dy is None:
        return o, None
    dy = dy.double()
    do = dy * p
    da = do @ w2
    dz = torch.cat([da * u * s * (1 + g * (1 - s)), da * g * s], 1)
    return o, (dz @ w1, (dy * o).sum(1), dz.t() @ x, do.t() @ a)


def exact(case, seed):
    c, d = case, _inputs(case, seed)
    if c["kind"] == "gate":
        return {"logits": d["X"].double() @ d["Wr"].double().t()}
    if c["kind"] == "router":
        return _exact_router(c, d)
    T, k, E, h, f = c["T"], c["k"], c["E"], c["h"], c["f"]
    sel, prob = _route(c, d["logits"], d.get("bias"))
    idx = d["idx"].long() if "idx" in d else sel
    align = 128 if c["recipe"] in ("fp8", "mxfp8") else 1
    flat = idx.flatten()
    counts = torch.bincount(flat, minlength=E)
    offsets = torch.zeros(E + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum((counts + align - 1) // align * align, 0)
    order = torch.argsort(flat, stable=True)
    first = torch.cumsum(counts, 0) - counts
    row_of = torch.empty(T * k, dtype=torch.int64, device="cuda")
    row_of[order] = torch.arange(T * k, device="cuda") - first[flat[order]] + offsets[flat[order]]
    f64 = dict(dtype=torch.float64, device="cuda")
    train = c["kind"] == "step"
    out = {"idx": sel.to(torch.int32), "prob": prob, "row_of": row_of.to(torch.int32).view(T, k),
           "offsets": offsets.to(torch.int32), "Y": torch.zeros((T, h), **f64)}
    if train:
        out.update(dX=torch.zeros((T, h), **f64), dprob=torch.zeros(T * k, **f64), dW1=torch.zeros((E, 2 * f, h), **f64),
                   dW2=torch.zeros((E, h, f), **f64))
    bounds = [0] + torch.cumsum(counts, 0).tolist()
    for e in range(E):
        pairs = order[bounds[e]:bounds[e + 1]]
        if not len(pairs):
            continue
        tok = pairs // k
        p = prob.flatten()[pairs, None]
        o, g = _mlp(d["X"][tok], d["W1"][e], d["W2"][e], p, d["dY"][tok] if train else None)
        out["Y"].index_add_(0, tok, p * o)
        if train:
            out["dX"].index_add_(0, tok, g[0])
            out["dprob"][pairs] = g[1]
            out["dW1"][e], out["dW2"][e] = g[2], g[3]
    if c["shared_f"]:
        o, g = _mlp(d["X"], d["Ws1"], d["Ws2"], 1.0, d["dY"] if train else None)
        out["Y"] += o
        if train:
            out["dX"] += g[0]
            out["dWs1"], out["dWs2"] = g[2], g[3]
    if train:
        out["dprob"] = out["dprob"].view(T, k)
    return out
