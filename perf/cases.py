"""Performance cases of the DeaMoE decode layer.

A case is one decode step's worth of work as a serving loop hands it over: one
call of the whole layer (router, plan, expert stages, combine) on a batch of T
tokens, with weights, workspace and output buffers in hand.  The layer shapes
are the presets of `paper_2608_14385_amd.workloads`; T spans the batches a
decode step can have (1 to 128).

The router weights and tokens lie on a grid on which every logit is exact in
fp32 whatever the order of its sum, so two correct implementations select the
same experts and only the arithmetic of the experts separates them.
"""
from __future__ import annotations

import functools
import math

import torch

from paper_2608_14385_amd import deamoe as D
from paper_2608_14385_amd import workloads as W

MAX_TOKENS = 128   # the batch a server sizes its workspace for


def _case(name, preset, tokens, bias=False, routing=False, entry="layer", sigma="silu"):
    return {"name": name, "preset": preset, "tokens": tokens, "bias": bias, "routing": routing,
            "entry": entry, "sigma": sigma}


def listed():
    return [
        # the smallest call: a tiny fp32 layer, launches and latency only
        _case("tiny_f32_t4", "tiny_f32", 4),
        # 7B-class layer with a shared expert: one user; a handful of users
        # through the entry point that takes no workspace; a busy server with
        # a ragged batch
        _case("7b_t1", "7b_bf16", 1),
        _case("7b_t16", "7b_bf16", 16, entry="noalloc"),
        _case("7b_t61", "7b_bf16", 61),
        # DeepSeek-V3-shaped layer: one user, the usual batch (with the
        # routing returned, as a server that tracks expert load asks for it),
        # the largest batch of the latency sweep
        _case("dsv3_t1", "dsv3_bf16", 1),
        _case("dsv3_t16", "dsv3_bf16", 16, routing=True),
        _case("dsv3_t64", "dsv3_bf16", 64),
        # the same with popular departments, at the largest batch there is
        _case("dsv3_skew_t128", "dsv3_skew", 128, bias=True),
        # the same with fp8 block-scaled weights, a ragged batch
        _case("dsv3_fp8_t45", "dsv3_fp8", 45),
        # the paper's FACTORED form (rows of its Table 1): a small model, the
        # large one at the usual batch, a middle one at a large batch
        _case("base7b_factored_t16", "base7b_factored", 16),
        _case("dsv3_factored_t16", "dsv3_factored", 16),
        _case("qwen3_factored_t64", "qwen3_factored", 64),
    ]


def draw(rng):
    largest = max(work(c)["bytes"] for c in listed())
    while True:
        preset = rng.choice(("tiny_f32", "7b_bf16", "7b_bf16", "dsv3_bf16", "dsv3_bf16", "dsv3_skew",
                             "dsv3_fp8", "dsv3_fp8", "base7b_factored", "qwen3_factored",
                             "dsv2_factored", "dsv3_factored"))
        tokens = min(MAX_TOKENS, int(2.0 ** rng.uniform(0.0, 7.0)))
        cfg = W.PRESETS[preset].layer
        sigma = "silu"
        if cfg.form == "factored" and rng.random() < 0.25:
            sigma = rng.choice(("none", "gelu", "rmsnorm"))
        case = {"preset": preset, "tokens": tokens, "bias": preset == "dsv3_skew",
                "routing": rng.random() < 0.25, "entry": "layer", "sigma": sigma}
        if work(case)["bytes"] <= largest:
            return case


def _config(case):
    return W.PRESETS[case["preset"]].layer.replace(sigma=case["sigma"])


def _inputs(case, seed):
    """Weights, tokens and the optional router bias, from the seed alone."""
    cfg = _config(case)
    w = W.make_weights(cfg, seed, device="cuda", gate_exact=True)
    x = W.make_tokens(cfg, case["tokens"], seed, device="cuda", gate_exact=True)
    bias = W.make_zipf_bias(cfg, seed).cuda() if case["bias"] else None
    return cfg, w, x, bias


def prepare(case, seed):
    cfg, w, x, bias = _inputs(case, seed)
    T = case["tokens"]
    state = {"entry": case["entry"], "x": x, "bias": bias, "y": torch.empty_like(x),
             "routing": D.Routing.alloc(cfg, T) if case["routing"] else None}
    if case["entry"] == "noalloc":
        state.update(c=D.make_config(cfg, MAX_TOKENS), weights=w, W=D.make_weights(w))
    else:
        state["layer"] = D.Layer(cfg, w, MAX_TOKENS)
    return state


def run(state):
    if state["entry"] == "noalloc":
        D.deamoe_layer_forward_noalloc(state["c"], state["x"], state["W"], state["y"],
                                       router_bias=state["bias"], routing=state["routing"])
    else:
        state["layer"](state["x"], router_bias=state["bias"], routing=state["routing"],
                       y=state["y"])
    if state["routing"] is None:
        return state["y"]
    return {"y": state["y"], **state["routing"].tensors}


# ------------------------------------------------------------- work of a pass


@functools.lru_cache(maxsize=None)
def _touched(n, m, k, kdept, T, zipf):
    """Mean departments, experts and (token, department) pairs a batch touches:
    logits of the drawn inputs are standard normal (plus the skew's bias)."""
    g = torch.Generator().manual_seed(1)
    E, reps = n // m, 8
    depts = exps = pairs = 0.0
    for _ in range(reps):
        l = torch.randn(T, n, generator=g)
        if zipf:
            wj = torch.arange(1, m + 1, dtype=torch.float32).pow(-1.2)
            l = l + torch.log(wj / wj.sum()).repeat_interleave(E)
        if kdept:
            gs = l.view(T, m, E).amax(-1)
            keep = torch.zeros(T, m, dtype=torch.bool)
            keep.scatter_(1, gs.topk(kdept, dim=1).indices, True)
            l = l.masked_fill(~keep.repeat_interleave(E, dim=1), -math.inf)
        ids = l.topk(k, dim=1).indices
        dm = torch.zeros(T, m, dtype=torch.bool).scatter_(1, ids // E, True)
        exps += ids.unique().numel() / reps
        depts += dm.any(0).sum().item() / reps
        pairs += dm.sum().item() / reps
    return depts, exps, pairs


def work(case):
    cfg, T = _config(case), case["tokens"]
    h, d, p, e = cfg.hidden, cfg.d_shared, cfg.d_private, cfg.d_shared_expert
    depts, exps, pairs = _touched(cfg.n_experts, cfg.n_depts, cfg.top_k, cfg.top_k_dept, T,
                                  case["bias"])
    wb = {"f32": 4, "bf16": 2, "fp8": 1}[cfg.w_dtype]
    ab = {"f32": 4, "bf16": 2}[cfg.act_dtype]

    def mats(r, c):   # three matrices, with fp8 their block scales
        return 3 * (r * c * wb + (-(-r // 128) * -(-c // 128) * 4 if cfg.w_dtype == "fp8" else 0))
    priv = (d, d) if cfg.form == "factored" else (p, h)
    nbytes = (cfg.n_experts * h * ab + 2 * T * h * ab + depts * mats(d, h) + exps * mats(*priv) +
              (mats(e, h) if e else 0))
    flops = 2 * (T * cfg.n_experts * h + 3 * pairs * d * h + 3 * T * cfg.top_k * priv[0] * priv[1] +
                 3 * T * e * h)
    return {"bytes": int(nbytes), "flops": int(flops)}


# -------------------------------------------------------------- correct results


def tolerance(case):
    """About four times the distance from 64 bits seen over the ranges: 2.4e-3
    (largest 1.0e-2) from the bf16 roundings of the gate/up outputs and of y,
    3.8e-3 (1.9e-2) with the interface vectors of the FACTORED form, 4.3e-7
    (1.7e-6) from the sums of the fp32 layer."""
    cfg = _config(case)
    if cfg.act_dtype == "f32":
        return {"rel": 1.7e-6, "max": 7e-6}
    return {"rel": 1.5e-2, "max": 8e-2} if cfg.form == "factored" else {"rel": 1e-2, "max": 4e-2}


def _sigma(v, kind):
    if kind == "silu":
        return v * torch.sigmoid(v)
    if kind == "gelu":
        return 0.5 * v * (1.0 + torch.erf(v * math.sqrt(0.5)))
    if kind == "rmsnorm":
        return v / torch.sqrt((v * v).mean(-1, keepdim=True) + 1e-6)
    return v


def _swiglu(x, g, u):
    a = x @ g.T
    return a * torch.sigmoid(a) * (x @ u.T)


def exact(case, seed):
    cfg, w, x, bias = _inputs(case, seed)
    T, n, m, k, E = case["tokens"], cfg.n_experts, cfg.n_depts, cfg.top_k, cfg.experts_per_dept
    dev = x.device

    def mat(key, i=None):
        t = w[key] if i is None else w[key][i]
        if cfg.w_dtype != "fp8":
            return t.double()
        s = w[key + "_scale"] if i is None else w[key + "_scale"][i]
        s = s.double().repeat_interleave(128, 0).repeat_interleave(128, 1)
        return t.view(torch.float8_e4m3fn).float().double() * s[:t.shape[0], :t.shape[1]]

    x64 = x.double()
    # the logits are exact in fp32 up to the bias, which is one fp32 addition
    logits = (x64 @ w["router"].double().T).float()
    if bias is not None:
        logits = logits + bias
    l = logits.double()
    sel = l
    if cfg.top_k_dept:   # departments by their best logit, ties to the lower id
        gs = l.view(T, m, E).amax(-1)
        keep = torch.zeros(T, m, dtype=torch.bool, device=dev)
        kept = torch.sort(gs, dim=1, descending=True, stable=True).indices[:, :cfg.top_k_dept]
        keep.scatter_(1, kept, True)
        sel = l.masked_fill(~keep.repeat_interleave(E, dim=1), -math.inf)
    ids = torch.sort(sel, dim=1, descending=True, stable=True).indices[:, :k]
    picked = l.gather(1, ids)
    if cfg.score == "softmax":
        p = torch.softmax(picked, 1) if cfg.renorm else torch.softmax(l, 1).gather(1, ids)
    else:
        p = torch.sigmoid(picked)
        if cfg.renorm:
            p = p / p.sum(1, keepdim=True)
    p = p * cfg.route_scale
    pe = torch.zeros(T, n, dtype=torch.float64, device=dev).scatter_(1, ids, p)
    has_e = torch.zeros(T, n, dtype=torch.bool, device=dev).scatter_(1, ids, True)
    has_d = has_e.view(T, m, E).any(-1)
    pd = pe.view(T, m, E).sum(-1)

    y = torch.zeros(T, cfg.hidden, dtype=torch.float64, device=dev)
    exps = has_e.any(0).nonzero().flatten().tolist()
    for j in has_d.any(0).nonzero().flatten().tolist():
        t = has_d[:, j].nonzero().flatten()
        if cfg.form == "slice":
            a = _swiglu(x64[t], mat("dept_gate", j), mat("dept_up", j))
            y[t] += pd[t, j, None] * (a @ mat("dept_down", j).T)
            continue
        g = torch.zeros(T, cfg.d_shared, dtype=torch.float64, device=dev)
        u, z = torch.zeros_like(g), torch.zeros_like(g)
        g[t] = _sigma(x64[t] @ mat("dept_gate", j).T, cfg.sigma)
        u[t] = _sigma(x64[t] @ mat("dept_up", j).T, cfg.sigma)
        for i in [i for i in exps if i // E == j]:
            ti = has_e[:, i].nonzero().flatten()
            v = g[ti] @ mat("priv_gate", i).T
            v = v * torch.sigmoid(v) * (u[ti] @ mat("priv_up", i).T)
            z[ti] += pe[ti, i, None] * _sigma(v @ mat("priv_down", i).T, cfg.sigma)
        y += z @ mat("dept_down", j).T
    if cfg.form == "slice" and cfg.d_private:
        for i in exps:
            t = has_e[:, i].nonzero().flatten()
            a = _swiglu(x64[t], mat("priv_gate", i), mat("priv_up", i))
            y[t] += pe[t, i, None] * (a @ mat("priv_down", i).T)
    if cfg.d_shared_expert:
        y += _swiglu(x64, mat("se_gate"), mat("se_up")) @ mat("se_down").T
    if not case["routing"]:
        return y

    i32 = torch.int32
    tok_depts = torch.full((T, k), -1, dtype=i32, device=dev)
    tok_dept_w = torch.zeros(T, k, dtype=torch.float64, device=dev)
    for t in range(T):
        js = has_d[t].nonzero().flatten()
        tok_depts[t, :len(js)] = js.to(i32)
        tok_dept_w[t, :len(js)] = pd[t, js]

    def csr(member):   # counts, offsets, ascending tokens (the unused tail keeps its fill)
        count = member.sum(0)
        offset = torch.cat([count.new_zeros(1), count.cumsum(0)])
        toks = torch.full((T * k,), -7, dtype=i32, device=dev)
        used = member.T.nonzero()[:, 1]
        toks[:len(used)] = used.to(i32)
        return count.to(i32), offset.to(i32), toks
    dc, do, dt = csr(has_d)
    ec, eo, et = csr(has_e)
    return {"y": y, "topk_ids": ids.to(i32), "topk_w": p, "tok_depts": tok_depts,
            "tok_dept_w": tok_dept_w, "tok_ndept": has_d.sum(1).to(i32), "dept_count": dc,
            "dept_offset": do, "dept_tokens": dt, "exp_count": ec, "exp_offset": eo,
            "exp_tokens": et, "logits": l}
