"""The workloads this library's speed is judged on, through its public entry points.

A case names one of the ways a program uses the library and the layer's shape:

  layer    one call of moe_layer_forward: inference, prefill or decode
  train    moe_layer_forward followed by moe_layer_backward: one layer of a training step
  experts  moe_grouped_ffn followed by moe_grouped_ffn_backward on rows that are already in expert
           order: a program that routes and exchanges the rows itself
  dispatch moe_route, moe_permute and moe_combine called one by one: a program with its own
           expert kernels between them

Shapes are those of ``paper_2607_18631_amd.workloads`` (or cuts of them) and, where noted, generic
odd ones.  Every input is drawn on the GPU from the seed with the distributions of
``workloads``: N(0, 1) token rows, weights scaled by 1/sqrt(fan-in), and a Zipf router bias where
the case is skewed.
"""
import math

import numpy as np
import torch

from paper_2607_18631_amd import moe
from paper_2607_18631_amd.workloads import GATE_SIGMOID, GATE_SOFTMAX, MoEShape, zipf_bias

BF16 = torch.bfloat16


def _case(kind, T, d, E, top_k, F, E_local, *, e_begin=0, F_shared=0, gate=GATE_SOFTMAX, n_group=1, topk_group=1,
          renormalize=1, routed_scale=1.0, expert_capacity=0, zipf=0.0, router_std=1.0):
    """router_std is in units of 1/sqrt(d)."""
    return {"kind": kind, "T": T, "d": d, "E": E, "top_k": top_k, "F": F, "E_local": E_local, "e_begin": e_begin,
            "F_shared": F_shared, "gate": gate, "n_group": n_group, "topk_group": topk_group,
            "renormalize": renormalize, "routed_scale": routed_scale, "expert_capacity": expert_capacity,
            "zipf": zipf, "router_std": router_std}


def listed():
    dsv3 = dict(d=7168, E=256, top_k=8, F=2048, E_local=32, F_shared=2048, gate=GATE_SIGMOID, n_group=8,
                topk_group=4, routed_scale=2.5)
    crossover = dict(d=2048, E=64, top_k=2, F=1408, E_local=8)
    cases = {
        # the smallest layer: launch count and latency decide
        "tiny_layer": _case("layer", T=256, d=512, E=8, top_k=2, F=1024, E_local=8, router_std=0.02 * 512 ** 0.5),
        # one decode step of an expert-parallel rank: a stream of the active experts' weights
        "decode_k2": _case("layer", T=64, d=7168, E=384, top_k=8, F=2048, E_local=48, F_shared=2048,
                           gate=GATE_SIGMOID),
        # a decode step in the static capacity layout that graph-captured serving uses
        "decode_masked": _case("layer", T=32, expert_capacity=8, **dsv3),
        # a small batch on a small rank share (the kernel-crossover shape, 16 tokens per expert)
        "small_batch": _case("layer", T=512, **crossover),
        # prefill of a DeepSeek-V3-shaped rank share (the benchmark's workload)
        "prefill_dsv3": _case("layer", T=8192, **dsv3),
        # prefill with few wide experts, all on one device
        "prefill_mixtral": _case("layer", T=4096, d=4096, E=8, top_k=2, F=14336, E_local=8),
        # prefill with many narrow experts and an uneven load
        "prefill_skewed": _case("layer", T=16384, d=2048, E=128, top_k=8, F=768, E_local=128, zipf=1.2,
                                router_std=2.0),
        # odd sizes: hidden and expert widths that are no multiple of a tile, a batch of odd length, a
        # shared expert of another width, an expert slice from the middle
        "prefill_ragged": _case("layer", T=3001, d=2040, E=40, top_k=5, F=1000, E_local=24, e_begin=9, F_shared=264,
                                gate=GATE_SIGMOID, renormalize=0),
        # one layer of a training step at the benchmark's shape
        "train_dsv3": _case("train", T=8192, **dsv3),
        # the same on a small rank share and a short batch
        "train_small": _case("train", T=2048, **crossover),
        # the expert MLP alone, forward and backward, on long segments
        "experts_long": _case("experts", T=32768, **crossover),
        # routing, permutation and combine around somebody else's expert kernels
        "dispatch_dsv3": _case("dispatch", T=8192, **dsv3),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _width(rng, lo, hi):
    """A hidden or expert width: usually a multiple of 128, sometimes any multiple of 8."""
    step = rng.choice([128, 128, 64, 8])
    return max(step, int(_log_uniform(rng, lo, hi) / step) * step)


def draw(rng):
    limit = work(_case("train", T=8192, d=7168, E=256, top_k=8, F=2048, E_local=32, F_shared=2048))["flops"] / 2
    while True:
        kind = rng.choice(["layer", "layer", "layer", "train", "train", "experts", "dispatch"])
        E = rng.choice([8, 16, 32, 40, 64, 96, 128, 160, 256, 384])
        top_k = rng.choice([k for k in (1, 2, 2, 4, 6, 8, 8) if 2 * k <= E])
        gate = rng.choice([GATE_SOFTMAX, GATE_SIGMOID])
        n_group, topk_group = 1, 1
        if gate == GATE_SIGMOID and rng.random() < 0.4:
            n_group = rng.choice([g for g in (2, 4, 8) if E // g >= 2])
            topk_group = rng.randint(max(1, -(-top_k * n_group // E)), n_group)
        E_local = max(1, E // rng.choice([1, 1, 2, 4, 8]))
        F = _width(rng, 256, 8192)
        T = int(_log_uniform(rng, 1, 16385))
        C = rng.randint(1, T) if kind == "layer" and T <= 256 and rng.random() < 0.3 else 0
        c = _case(kind, T=T, d=_width(rng, 512, 7168), E=E, top_k=top_k, F=F, E_local=E_local,
                  e_begin=rng.randint(0, E - E_local), F_shared=rng.choice([0, 0, F, _width(rng, 256, 4096)]), gate=gate,
                  n_group=n_group, topk_group=topk_group, renormalize=rng.choice([0, 1, 1]),
                  routed_scale=rng.choice([1.0, 2.5]), expert_capacity=C,
                  zipf=1.2 if gate == GATE_SOFTMAX and rng.random() < 0.3 else 0.0, router_std=rng.choice([1.0, 2.0]))
        w = work(c)
        resident = 6 * c["d"] * (c["E_local"] * c["F"] + c["F_shared"])       # bytes of expert weights
        if w["flops"] <= limit and w["bytes"] <= 6e9 and resident <= 4e9:
            return c


def _shape(case):
    keys = ("T", "d", "E", "top_k", "F", "E_local", "e_begin", "F_shared", "gate", "n_group", "topk_group",
            "renormalize", "routed_scale", "expert_capacity")
    return MoEShape(**{k: case[k] for k in keys})


def _inputs(case, seed):
    sh = _shape(case)
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(std, *size):
        return torch.empty(size, dtype=BF16, device="cuda").normal_(0.0, std, generator=g)

    T, d, F, Fs, El = sh.T, sh.d, sh.F, sh.F_shared, sh.E_local
    t = {"x": normal(1.0, T, d), "w_router": normal(case["router_std"] * d ** -0.5, sh.E, d)}
    t["bias"] = torch.from_numpy(zipf_bias(sh.E, case["zipf"], seed)).cuda() if case["zipf"] > 0 else None
    if case["kind"] != "dispatch":
        t["w13"], t["w2"] = normal(d ** -0.5, El, 2 * F, d), normal(F ** -0.5, El, d, F)
        t["ws13"] = normal(d ** -0.5, 2 * Fs, d) if Fs else None
        t["ws2"] = normal(Fs ** -0.5, d, Fs) if Fs else None
    if case["kind"] == "train":
        t["dout"] = normal(1.0, T, d)
    if case["kind"] == "experts":
        # rows of each expert: the loads of a batch under uniform routing
        rows = np.random.RandomState(seed % (1 << 32)).multinomial(_local_rows(case), [1.0 / El] * El)
        t["offsets"] = torch.from_numpy(np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)).cuda()
        n = int(rows.sum())
        t["x_perm"], t["dy_perm"] = normal(1.0, n, d), normal(1.0, n, d)
    if case["kind"] == "dispatch":
        t["y_perm"] = normal(1.0, sh.capacity, d)
        t["shared_y"] = normal(1.0, T, d) if Fs else None
    return sh, t


def _local_rows(case):
    """Expected (token, expert) pairs on this rank."""
    n = case["T"] * case["top_k"] * case["E_local"] / case["E"]
    if case["expert_capacity"] > 0:
        n = min(n, case["E_local"] * case["expert_capacity"])
    return max(1, round(n))


def _empty(dtype, *size):
    return torch.empty(size, dtype=dtype, device="cuda")


def prepare(case, seed):
    """Inputs, weights, outputs and workspaces of one layer, as a program holds them between calls."""
    sh, s = _inputs(case, seed)
    s["kind"] = case["kind"]
    T, d, F, Fs, El, k = sh.T, sh.d, sh.F, sh.F_shared, sh.E_local, sh.top_k
    if case["kind"] in ("layer", "train"):
        s["out"] = _empty(BF16, T, d)
        s["ws"] = moe.alloc_workspace(sh, moe.MOE_WS_LAYER)
    if case["kind"] == "train":
        s["ws_bwd"] = moe.alloc_workspace(sh, moe.MOE_WS_LAYER_BWD)
        s["dx"], s["dw_router"] = _empty(BF16, T, d), _empty(BF16, sh.E, d)
        s["dws13"], s["dws2"] = (_empty(BF16, 2 * Fs, d), _empty(BF16, d, Fs)) if Fs else (None, None)
    if case["kind"] == "experts":
        # the entry points take buffers of the shape's capacity; a program that holds n rows describes
        # them as n tokens with one local expert choice each
        n = s["x_perm"].shape[0]
        sh = sh.replace(T=n, top_k=1, F_shared=0, n_group=1, topk_group=1)
        s["y_perm"], s["dx_perm"] = _empty(BF16, n, d), _empty(BF16, n, d)
        s["ws"], s["ws_bwd"] = moe.alloc_workspace(sh, moe.MOE_WS_FFN), moe.alloc_workspace(sh, moe.MOE_WS_FFN_BWD)
    if case["kind"] in ("train", "experts"):
        s["dw13"], s["dw2"] = _empty(BF16, El, 2 * F, d), _empty(BF16, El, d, F)
    if case["kind"] == "dispatch":
        i32 = torch.int32
        s["topk_idx"], s["topk_w"] = _empty(i32, T, k), _empty(torch.float32, T, k)
        s["counts"], s["offsets"] = _empty(i32, El), _empty(i32, El + 1)
        # rows past the routed ones are not written: they start defined
        s["row_token"] = torch.zeros(sh.capacity, dtype=i32, device="cuda")
        s["x_perm"] = torch.zeros(sh.capacity, d, dtype=BF16, device="cuda")
        s["slot_row"], s["out"] = _empty(i32, T, k), _empty(BF16, T, d)
        s["ws_route"] = moe.alloc_workspace(sh, moe.MOE_WS_ROUTE)
        s["ws_permute"] = moe.alloc_workspace(sh, moe.MOE_WS_PERMUTE)
    s["shape"] = sh
    return s


def run(s):
    sh, kind = s["shape"], s["kind"]
    if kind == "experts":
        moe.moe_grouped_ffn(sh, s["x_perm"], s["offsets"], s["w13"], s["w2"], s["y_perm"], s["ws"])
        moe.moe_grouped_ffn_backward(sh, s["x_perm"], s["offsets"], s["w13"], s["w2"], s["dy_perm"], s["dx_perm"],
                                     s["dw13"], s["dw2"], s["ws_bwd"])
        return {n: s[n] for n in ("y_perm", "dx_perm", "dw13", "dw2")}
    if kind == "dispatch":
        moe.moe_route(sh, s["x"], s["w_router"], s["bias"], s["topk_idx"], s["topk_w"], None, s["ws_route"])
        moe.moe_permute(sh, s["topk_idx"], s["x"], s["counts"], s["offsets"], s["row_token"], s["slot_row"],
                        s["x_perm"], s["ws_permute"])
        moe.moe_combine(sh, s["y_perm"], s["slot_row"], s["topk_w"], s["shared_y"], s["out"])
        return {n: s[n] for n in ("topk_idx", "topk_w", "counts", "offsets", "slot_row", "x_perm", "out")}
    moe.moe_layer_forward(sh, s["x"], s["w_router"], s["bias"], s["w13"], s["w2"], s["ws13"], s["ws2"], s["out"],
                          s["ws"])
    if kind == "layer":
        return {"out": s["out"]}
    moe.moe_layer_backward(sh, s["x"], s["w_router"], s["bias"], s["w13"], s["w2"], s["ws13"], s["ws2"], s["dout"],
                           s["ws"], s["dx"], s["dw_router"], s["dw13"], s["dw2"], s["dws13"], s["dws2"], s["ws_bwd"])
    names = ["out", "dx", "dw_router", "dw13", "dw2"] + (["dws13", "dws2"] if sh.F_shared else [])
    return {n: s[n] for n in names}


def work(case):
    T, d, E, F, Fs, El, k = (case[n] for n in ("T", "d", "E", "F", "F_shared", "E_local", "top_k"))
    n = _local_rows(case)
    rows = 2.0 * d                                       # bytes of one row of d values
    router = {"bytes": 2.0 * E * d, "flops": 2.0 * T * E * d}
    # experts with at least one row under uniform routing
    active = El * (1.0 - (1.0 - k / E) ** T) if case["zipf"] == 0 else El
    weights, shared = 6.0 * d * F, 6.0 * d * Fs
    mlp = 6.0 * d * (F * n + Fs * T)
    if case["kind"] == "dispatch":
        # token rows read once for the logits and the copy, the rows written, the rows combined
        b = T * rows + router["bytes"] + 2 * n * rows + T * rows * (2 if Fs else 1) + 16.0 * T * k
        return {"bytes": b, "flops": router["flops"]}
    if case["kind"] == "experts":
        # rows in, out, their gradients in and out; weights in, their gradients out
        return {"bytes": 4 * n * rows + active * weights + El * weights, "flops": 18.0 * d * F * n}
    fwd = {"bytes": 2 * T * rows + router["bytes"] + active * weights + shared, "flops": router["flops"] + mlp}
    if case["kind"] == "layer":
        return fwd
    return {"bytes": fwd["bytes"] + 2 * T * rows + router["bytes"] + El * weights + shared,
            "flops": 3 * router["flops"] + 3 * mlp}


def tolerance(case):
    # bf16 results (0.17% rms) of bf16 intermediates; gradients pass up to five such roundings.  A
    # routing decision on a rounding tie may fall the other way.
    if case["kind"] == "dispatch":
        return {"rel": 6e-3, "differ": 1e-3}
    return {"rel": 1e-2 if case["kind"] == "layer" else 1.4e-2}


# ---- the same results in 64 bits, in plain torch ----
def _mlp(x, w13, w2):
    F = w2.shape[1]
    return (torch.nn.functional.silu(x @ w13[:F].t()) * (x @ w13[F:].t())) @ w2.t()


def _route64(sh, x, w_router, bias):
    """(chosen experts, their gates); the gates are differentiable, the choice is not."""
    logits = x @ w_router.t()
    keys = logits.sigmoid() if sh.gate == GATE_SIGMOID else logits if bias is None else logits + bias
    score = keys.detach()
    if sh.n_group > 1:
        grouped = score.view(sh.T, sh.n_group, -1)
        best = grouped.topk(2, dim=2).values.sum(2).topk(sh.topk_group, dim=1).indices
        keep = torch.zeros(sh.T, sh.n_group, dtype=torch.bool, device=x.device).scatter_(1, best, True)
        score = grouped.masked_fill(~keep[:, :, None], -math.inf).view(sh.T, sh.E)
    idx = score.topk(sh.top_k, dim=1).indices
    chosen = keys.gather(1, idx)
    if sh.gate == GATE_SIGMOID:
        gates = chosen / chosen.sum(1, keepdim=True) if sh.renormalize else chosen
    else:
        gates = chosen.softmax(1) if sh.renormalize else keys.softmax(1).gather(1, idx)
    return idx, gates * sh.routed_scale


def _kept(sh, idx, e):
    """(tokens, slots) of expert e's rows, ascending by token, cut at the capacity."""
    tok, slot = (idx == e).nonzero(as_tuple=True)
    C = sh.expert_capacity if sh.expert_capacity > 0 else tok.numel()
    return tok[:C], slot[:C]


def exact(case, seed):
    sh, t = _inputs(case, seed)
    kind = case["kind"]
    wide = {n: v.double() for n, v in t.items() if v is not None and v.is_floating_point() and n not in ("w13", "w2")}
    if kind == "experts":
        res = {n: [] for n in ("y_perm", "dx_perm", "dw13", "dw2")}
        ends = t["offsets"].tolist()
        for e in range(sh.E_local):
            a, b = ends[e], ends[e + 1]
            leaves = [v.double().requires_grad_() for v in (t["x_perm"][a:b], t["w13"][e], t["w2"][e])]
            y = _mlp(*leaves)
            grads = torch.autograd.grad(y, leaves, wide["dy_perm"][a:b])
            for n, v in zip(res, (y.detach(), *grads)):
                res[n].append(v)
        return {n: (torch.stack if n in ("dw13", "dw2") else torch.cat)(v) for n, v in res.items()}
    train = kind == "train"
    x, w_router = wide["x"].requires_grad_(train), wide["w_router"].requires_grad_(train)
    idx, gates = _route64(sh, x, w_router, wide.get("bias"))
    local = [(e, *_kept(sh, idx, sh.e_begin + e)) for e in range(sh.E_local)]
    out = torch.zeros(sh.T, sh.d, dtype=torch.float64, device="cuda")
    if kind == "dispatch":
        start = 0
        x_perm = torch.zeros(sh.capacity, sh.d, dtype=torch.float64, device="cuda")
        for _, tok, slot in local:
            end = start + tok.numel()
            x_perm[start:end] = x[tok]
            out.index_add_(0, tok, gates[tok, slot][:, None] * wide["y_perm"][start:end])
            start = end
        if sh.F_shared:
            out += wide["shared_y"]
        return {"topk_idx": None, "topk_w": gates, "counts": None, "offsets": None, "slot_row": None,
                "x_perm": x_perm, "out": out}
    shared = [wide[n].requires_grad_(train) for n in ("ws13", "ws2")] if sh.F_shared else []
    experts = []
    for e, tok, slot in local:
        w13, w2 = (t[n][e].double().requires_grad_(train) for n in ("w13", "w2"))
        out = out.index_add(0, tok, gates[tok, slot][:, None] * _mlp(x[tok], w13, w2))
        if train:
            experts += [w13, w2]
    if shared:
        out = out + _mlp(x, *shared)
    if not train:
        return {"out": out}
    grads = torch.autograd.grad(out, [x, w_router, *experts, *shared], wide["dout"])
    n = 2 + len(experts)
    res = {"out": out.detach(), "dx": grads[0], "dw_router": grads[1], "dw13": torch.stack(grads[2:n:2]),
           "dw2": torch.stack(grads[3:n:2])}
    if shared:
        res["dws13"], res["dws2"] = grads[n:]
    return res
