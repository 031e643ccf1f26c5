"""The workloads this layer is timed on: what they are, how their inputs are made, and one pass of each.

A case is one layer (tokens, widths, two-level router, capacity, storage type, activation, options) and one way
of using it:

  infer   one forward pass through smile_layer_forward without expert buffers (the serving form);
  steps   the same forward pass as six separate calls with materialised expert buffers, for programs that put
          work of their own between the steps;
  train   a training step: the forward pass that keeps what the backward pass needs (with `saved`, also the hidden
          activation and its pre-activation), then smile_layer_backward.

Everything a program keeps between calls -- weights, ctx, buffers, the argument blocks -- is made by prepare();
run() only makes the library calls.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2212_05191_amd import binding as B

ALPHA = BETA = 0.005       # loss coefficients of the paper's training runs
DLOSS = 1.0


def _case(name, mode, T, d_model, d_ff, n_groups, m_local, capacity_factor, dtype, act="gelu", skew=False,
          expert_bias=False, group_factor=0.0, saved=True):
    c = dict(name=name, mode=mode, T=T, d_model=d_model, d_ff=d_ff, n_groups=n_groups, m_local=m_local,
             capacity_factor=capacity_factor, dtype=dtype, act=act, skew=skew, expert_bias=expert_bias,
             group_factor=group_factor, saved=saved)
    return c if name else {k: v for k, v in c.items() if k != "name"}


def listed():
    return [
        # The smallest layer of the benchmark set (single precision, ReLU): nothing but launches and latency.
        _case("infer_tiny_f32", "infer", 512, 64, 128, 2, 2, 1.25, "f32", "relu"),
        # One sequence of 128 tokens through a 16-expert layer of the base width: a handful of rows per expert, every
        # weight read for them.  Capacity factor 2, the paper's evaluation setting.
        _case("infer_one_sequence", "infer", 128, 768, 3072, 2, 8, 2.0, "bf16"),
        # The base layer on its micro-batch (8 x 1024 tokens): a few hundred rows per expert.
        _case("infer_base", "infer", 8192, 768, 3072, 2, 8, 1.0, "bf16"),
        # A batch that divides by nothing, in half precision, with expert biases and a first-hop buffer limit: the
        # last batch of a data set, variable-length input, an odd group layout.
        _case("infer_ragged_f16", "infer", 5003, 960, 3840, 3, 5, 1.25, "f16", "relu", expert_bias=True,
              group_factor=1.25),
        # The wider model (1024 / 4096) with 64 experts.
        _case("infer_large", "infer", 16384, 1024, 4096, 8, 8, 1.25, "bf16"),
        # Many experts, routing-heavy: 16 groups of 8.
        _case("infer_many_experts", "infer", 32768, 768, 3072, 16, 8, 1.0, "bf16"),
        # The same experts behind the flat one-level router the paper compares against.
        _case("infer_flat_router", "infer", 32768, 768, 3072, 1, 128, 1.0, "bf16"),
        # The largest batch and expert count with a skewed router: drops, empty and overfull experts.
        _case("infer_skewed", "infer", 65536, 1024, 4096, 32, 8, 1.0, "bf16", skew=True),
        # Training steps: the base layer, ...
        _case("train_base", "train", 8192, 768, 3072, 2, 8, 1.0, "bf16"),
        # ... the widest model (1600 / 6400) with half-empty buffers, ...
        _case("train_wide", "train", 8192, 1600, 6400, 2, 8, 2.0, "bf16"),
        # ... and the largest batch with the skewed router, where the weight gradients are most of the bytes.
        _case("train_skewed", "train", 65536, 1024, 4096, 32, 8, 1.0, "bf16", skew=True),
        # Training in single precision, as done to check a model or a port of one.
        _case("train_f32", "train", 2048, 256, 1024, 2, 4, 1.25, "f32"),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _multiple(v, q, lo):
    return max(lo, int(round(v / q)) * q)


def _cost(c):
    """Time-like size of a case (seconds at nominal rates), to keep drawn cases within the listed ones."""
    w = work(c)
    return w["bytes"] / 8e12 + w["flops"] / (1e14 if c["dtype"] == "f32" else 2.5e15)


def draw(rng):
    most = {"f32": _cost(listed()[-1]), "f16": _cost(listed()[-2]), "bf16": _cost(listed()[-2])}
    while True:
        dtype = rng.choices(("bf16", "f16", "f32"), (65, 20, 15))[0]
        mode = rng.choices(("infer", "steps", "train"), (55, 10, 35))[0]
        q = 8 if dtype == "f32" else 64
        d = _multiple(_log_uniform(rng, 64, 512 if dtype == "f32" else 1600), q, 64)
        F = _multiple(d * rng.choice((2, 3, 4, 4, 4)), q, 64)
        # two levels of like size, or the flat router
        if rng.random() < 0.15:
            n, m = 1, int(round(_log_uniform(rng, 4, 128)))
        else:
            n, m = int(round(_log_uniform(rng, 2, 32))), rng.randint(2, 8)
        T = int(round(_log_uniform(rng, 32, 65536)))
        if rng.random() < 0.5:
            T = max(32, T // 32 * 32)      # whole sequences as often as odd remainders
        c = _case("", mode, T, d, F, n, m, rng.choice((1.0, 1.25, 1.5, 2.0)), dtype,
                  rng.choices(("gelu", "relu"), (75, 25))[0], skew=rng.random() < 0.25,
                  expert_bias=mode != "train" and rng.random() < 0.25,
                  group_factor=1.25 if n > 1 and rng.random() < 0.15 else 0.0, saved=rng.random() < 0.8)
        if _cost(c) <= most[dtype]:
            return c


def _capacities(case):
    """(rows per expert buffer, rows per first-hop buffer or 0)"""
    T, n, m = case["T"], case["n_groups"], case["m_local"]
    cap = B.smile_capacity(T, n * m, case["capacity_factor"])
    return cap, math.ceil(case["group_factor"] * T / n) if case["group_factor"] else 0


def prepare(case, seed):
    dev = "cuda:0"
    T, d, F, n, m = (case[k] for k in ("T", "d_model", "d_ff", "n_groups", "m_local"))
    N, st = n * m, B.torch_dtype(case["dtype"])
    cap, group_cap = _capacities(case)
    g = torch.Generator(device=dev).manual_seed(int(seed))

    def normal(*shape, std=1.0, dtype=st):
        return torch.empty(shape, dtype=dtype, device=dev).normal_(0.0, std, generator=g)

    s = {"mode": case["mode"]}
    s["desc"] = desc = B.make_desc(T, d, F, n, m, cap, case["dtype"], case["act"], ALPHA, BETA, group_cap)
    # activations of unit variance, weights with the BERT initialiser's standard deviation
    s["x"] = normal(T, d)
    s["w_inter"], s["w_intra"] = normal(n, d, std=0.02), normal(m, d, std=0.02)
    s["w1"], s["w2"] = normal(N, F, d, std=0.02), normal(N, d, F, std=0.02)
    s["b1"] = normal(N, F, std=0.02) if case["expert_bias"] else None
    s["b2"] = normal(N, d, std=0.02) if case["expert_bias"] else None
    s["bias_inter"] = s["bias_intra"] = None
    if case["skew"]:      # Zipf ranking over the groups, independent preferences inside each
        rank = torch.randperm(n, device=dev, generator=g).double() + 1.0
        s["bias_inter"] = (2.0 * rank ** -1.2).float()
        s["bias_intra"] = normal(n, m, std=0.5, dtype=torch.float32)
    s["workspace"] = torch.empty(B.smile_workspace_bytes(desc), dtype=torch.uint8, device=dev)
    s["ctx"] = B.Ctx(desc, s["workspace"])
    s["buf"] = B.alloc_buffers(desc, dev)
    s["io"] = B.make_io(s["x"], s["w_inter"], s["w_intra"], s["w1"], s["w2"], s["buf"], s["b1"], s["b2"],
                        s["bias_inter"], s["bias_intra"])
    if case["mode"] == "infer":
        s["io"].xe = s["io"].ye = None
    if case["mode"] == "train":
        s["dy"] = normal(T, d)
        s["h"] = s["pre"] = None
        if case["saved"]:
            s["h"], s["pre"] = torch.empty((N, cap, F), dtype=st, device=dev), torch.empty((N, cap, F), dtype=st, device=dev)
            s["io"].h_save, s["io"].pre_save = s["h"].data_ptr(), s["pre"].data_ptr()
        s["bwd"] = B.alloc_backward_buffers(desc, dev)
        s["bwd_workspace"] = torch.empty(B.smile_backward_workspace_bytes(desc), dtype=torch.uint8, device=dev)
        s["bwd_io"] = B.make_backward_io(s["x"], s["w_inter"], s["w_intra"], s["w1"], s["w2"], s["buf"], s["dy"],
                                         s["bwd"], s["bias_inter"], s["bias_intra"], s["h"], s["pre"])
    return s


def run(s):
    b = s["buf"]
    if s["mode"] == "steps":
        ctx = s["ctx"]
        B.smile_gate_logits(ctx, s["x"], s["w_inter"], s["w_intra"], b.logits_inter, b.logits_intra)
        B.smile_route_bilevel(ctx, b.logits_inter, b.logits_intra, s["bias_inter"], s["bias_intra"], b.group_idx,
                              b.local_idx, b.pos_in_group, b.slot, b.gate, b.p_top, b.q_top, b.group_count,
                              b.local_count, b.expert_count, b.kept_count, b.p_sum, b.q_sum)
        B.smile_dispatch(ctx, s["x"], b.group_idx, b.local_idx, b.slot, b.xe)
        B.smile_expert_ffn(ctx, b.xe, b.kept_count, s["w1"], s["b1"], s["w2"], s["b2"], b.ye)
        B.smile_combine(ctx, b.ye, b.group_idx, b.local_idx, b.slot, b.gate, b.y)
        B.smile_aux_loss(ctx, b.group_count, b.local_count, b.p_sum, b.q_sum, b.loss3)
    else:
        B.smile_layer_forward(s["ctx"], s["io"])
    out = {"y": b.y, "loss": b.loss3, "logits_inter": b.logits_inter, "logits_intra": b.logits_intra,
           "gate": b.gate, "p_top": b.p_top, "q_top": b.q_top, "p_sum": b.p_sum, "q_sum": b.q_sum,
           "group_idx": b.group_idx, "local_idx": b.local_idx, "pos_in_group": b.pos_in_group, "slot": b.slot,
           "group_count": b.group_count, "local_count": b.local_count, "expert_count": b.expert_count,
           "kept_count": b.kept_count}
    if s["mode"] == "train":
        B.smile_layer_backward(s["ctx"], s["bwd_io"], DLOSS, s["bwd_workspace"])
        w = s["bwd"]
        out.update(dx=w.dx, dw_inter=w.dw_inter, dw_intra=w.dw_intra, dw1=w.dw1, dw2=w.dw2)
    return out


def _expected_load(case):
    """Expected (kept rows over all experts, experts with at least one row) under prepare()'s inputs."""
    T, n, m = case["T"], case["n_groups"], case["m_local"]
    cap, group_cap = _capacities(case)
    p = np.full(n * m, 1.0 / (n * m))
    if case["skew"]:      # expert probabilities from a sample of router logits with the two biases
        r, sd = np.random.default_rng(7), 0.02 * math.sqrt(case["d_model"])
        a = sd * r.standard_normal((4096, n)) + 2.0 * np.arange(1.0, n + 1.0) ** -1.2
        pref = 0.5 * r.standard_normal((n, m))
        gi = a.argmax(1)
        e = gi * m + (sd * r.standard_normal((4096, m)) + pref[gi]).argmax(1)
        p = np.bincount(e, minlength=n * m) / 4096.0
    load = T * p
    if group_cap:
        per_group = load.reshape(n, m).sum(1, keepdims=True)
        load = (load.reshape(n, m) * np.minimum(1.0, group_cap / np.maximum(per_group, 1e-9))).ravel()
    # E[min(X, cap)] for X ~ Normal(load, load): the Poisson spread of an expert's arrivals
    sd = np.sqrt(np.maximum(load, 1e-9))
    z = (cap - load) / sd
    phi = np.exp(-0.5 * z * z) / math.sqrt(2 * math.pi)
    Phi = np.array([0.5 * (1 + math.erf(v / math.sqrt(2))) for v in z])
    kept = np.clip(load * Phi - sd * phi + cap * (1 - Phi), 0.0, np.minimum(load, cap))
    return float(kept.sum()), float((1 - np.exp(-load)).sum())


def work(case):
    T, d, F, n, m = (case[k] for k in ("T", "d_model", "d_ff", "n_groups", "m_local"))
    s = 4 if case["dtype"] == "f32" else 2
    kept, live = _expected_load(case)
    weights = 2.0 * d * F * s
    # tokens in, outputs out, the routing results, router weights, the weights of the experts that have rows
    nbytes = 2.0 * T * d * s + T * (4.0 * (n + m) + 28.0) + (n + m) * d * s + live * weights
    flops = 4.0 * kept * d * F + 2.0 * T * (n + m) * d
    if case["mode"] == "train":
        # upstream gradient in, token gradient, router and expert weight gradients out
        nbytes += 2.0 * T * d * s + (n + m) * d * 4.0 + n * m * weights
        flops += 8.0 * kept * d * F + 4.0 * T * (n + m) * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # sums in the storage type's working precision: fp32, or 16-bit operands and results with fp32 accumulation.
    # `differ`: top-1 ties may fall the other way where logits are summed in another order.
    return {"f32": {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}, "bf16": {"rel": 1e-2, "max": 0.1, "differ": 1e-3},
            "f16": {"rel": 2e-3, "max": 0.02, "differ": 1e-3}}[case["dtype"]]
