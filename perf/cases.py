"""The work a participant's program has the framework do, as measurable cases.

A case is one call sequence through the public entry points of
``paper_2508_19078_amd`` on one MoE layer (or a small stack of layers):

  eval     a layer's forward: route -> permute -> grouped SwiGLU -> combine
           (evaluation and generation with the fine-tuned model)
  train    a layer's fine-tuning step on one or more micro-batches: the forward,
           then combine backward -> grouped SwiGLU backward -> permute backward,
           optionally the router backward and the expert utilities
  profile  the quantised profiling pass over a stack of layers (QuantizedStack)
           with the activation frequencies it exists for
  merge    the once-per-round merge of a layer's least activated experts:
           quantise the router, histogram, frequencies, weighted merge
  cluster  the once-per-round layer-aware clustering: merge budget, then PCA
           and K-Means of every layer's non-tuning experts

Ranges (what ``draw`` spreads over): 1 to 32768 tokens, d from 128 to 4096 and I
from 64 to 2816 in multiples of 8, 4 to 128 experts, top-1 to top-8, none to two
shared experts, bf16 mostly and fp32, popularity from even to Zipf.
"""
import math

import torch

from paper_2508_19078_amd import api
from paper_2508_19078_amd.profiling import QuantizedStack

DEV = "cuda"
DT = {"bf16": torch.bfloat16, "f32": torch.float32}


# ------------------------------------------------------------------ cases ----

def _layer(kind, T, d, E, k, I, dtype="bf16", shared=0, merged=0, group=4, skew="normal", **more):
    """merged experts share slots in groups of `group`."""
    return dict(kind=kind, T=T, d=d, E=E, k=k, I=I, dtype=dtype, shared=shared, merged=merged, group=group,
                skew=skew, **more)


def listed():
    return [
        # the unit workload of the test suite: the smallest fine-tuning step, fp32, where launches count
        dict(_layer("train", 256, 128, 8, 2, 256, "f32", merged=4, group=2, skew="even", tune=6, micro=1, gates=True,
                    utility=True), name="train_tiny_f32"),
        # generation with the LLaMA-MoE-shaped layer: one token of each of 8 sequences
        dict(_layer("eval", 8, 4096, 16, 4, 688), name="eval_llama_8_tokens"),
        # one short prompt through the DeepSeek-MoE-shaped layer, a length off every tile
        dict(_layer("eval", 333, 2048, 64, 6, 1408, shared=2), name="eval_deepseek_333"),
        # a constrained participant: two micro-batches of 512 tokens with accumulated weight
        # gradients, the stack's merged layer (16 tuning experts)
        dict(_layer("train", 512, 2048, 64, 6, 1408, merged=24, tune=16, micro=2, gates=False, utility=False),
             name="train_deepseek_micro_512"),
        # the LLaMA-MoE-shaped layer's step (every expert tunes)
        dict(_layer("train", 4096, 4096, 16, 4, 688, tune=16, micro=1, gates=False, utility=False),
             name="train_llama_4096"),
        # the benchmark's layer: the DeepSeek-MoE-shaped step, with the router's share of dX and the utilities
        dict(_layer("train", 8192, 2048, 64, 6, 1408, shared=2, merged=32, tune=32, micro=1, gates=True, utility=True),
             name="train_deepseek_8192"),
        # the stress layer: 262144 rows, Zipf popularity
        dict(_layer("train", 32768, 4096, 64, 8, 1024, skew="zipf", tune=64, micro=1, gates=False, utility=False),
             name="train_stress_32768"),
        # fine-tuning in full precision, sizes off every tile
        dict(_layer("train", 1023, 1000, 16, 4, 616, "f32", shared=1, tune=16, micro=1, gates=True, utility=False),
             name="train_f32_1023"),
        # two layers of the DeepSeek-MoE-shaped stack's profiling pass
        dict(_layer("profile", 4096, 2048, 64, 6, 1408, layers=2), name="profile_deepseek_2x4096"),
        # the LLaMA-MoE-shaped layer profiled on a small local data set
        dict(_layer("profile", 777, 4096, 16, 4, 688, layers=1), name="profile_llama_777"),
        # the benchmark's layer merged from 8192 profiled tokens
        dict(_layer("merge", 8192, 2048, 64, 6, 1408, merged=32), name="merge_deepseek"),
        # four layers of the stack clustered (48 non-tuning experts each)
        dict(kind="cluster", layers=4, E=64, d=2048, I=1408, dtype="bf16", tune=16, r=8, classes=9,
             name="cluster_deepseek_4"),
    ]


def _spread(rng, lo, hi, step):
    """A multiple of `step` in [lo, hi], spread over its logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choices(("eval", "train", "profile", "merge", "cluster"), (5, 8, 3, 2, 1))[0]
    while True:
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        d, I = _spread(rng, 128, 4096, 8), _spread(rng, 64, 2816, 8)
        E = rng.choice((4, 8, 16, 24, 32, 48, 64, 64, 96, 128))
        es = 4 if dtype == "f32" else 2
        if kind == "cluster":
            E = min(E, 64)
            c = dict(kind=kind, layers=rng.randint(1, 8), E=E, d=d, I=I, dtype=dtype, tune=E // 4,
                     r=max(1, E // 8), classes=max(1, E // 8) + 1)
            if 3 * d * I * E * c["layers"] * es < 4e9 and (d * I * es) % 16 == 0:
                return c
            continue
        T, k = _spread(rng, 1, 32768, 1), rng.randint(1, min(8, E))
        skew = rng.choice(("normal", "normal", "even", "zipf"))
        shared = rng.choice((0, 0, 1, 2))
        if kind == "merge":
            c = _layer(kind, max(T, 16), d, E, k, I, dtype, 0, E // 2, rng.choice((2, E // 4 or 1)), skew)
        elif kind == "profile":
            if rng.random() < 0.8:
                dtype, d, I = "bf16", d // 16 * 16, max(64, I // 16 * 16)
            c = _layer(kind, T, d, E, k, I, dtype, shared, skew=skew, layers=rng.randint(1, 3))
        else:
            merged = rng.choice((0, 0, E // 2))
            c = _layer(kind, T, d, E, k, I, dtype, shared, merged, 2 if E < 8 else 4, skew)
            if kind == "train":
                s = E - merged + merged // c["group"]
                c.update(tune=rng.choice((s, max(1, s // 2))), micro=rng.choice((1, 1, 2)),
                         gates=rng.random() < 0.5, utility=rng.random() < 0.3)
        # no dearer than the largest listed case: its flops, and fp32 at a sixteenth of the bf16 rate
        w = work(c)
        if w["flops"] * (16 if dtype == "f32" else 1) < 1.5e13 and w["bytes"] < 8e9:
            return c


# ---------------------------------------------------------------- prepare ----

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std, dt):
    return torch.randn(shape, generator=g, device=DEV).mul_(std).to(dt)


def _bias(c, g):
    """The logit bias that skews the experts' popularity."""
    E = c["E"]
    if c["skew"] == "normal":
        return torch.randn(E, generator=g, device=DEV)
    if c["skew"] == "zipf":
        return -1.2 * torch.log(torch.randperm(E, generator=g, device=DEV).float() + 1)
    return torch.zeros(E, device=DEV)


def _experts(c, g, n):
    """W_gate, W_up [n, I, d] and W_down [n, d, I]."""
    d, I, dt = c["d"], c["I"], DT[c["dtype"]]
    return (_normal(g, (n, I, d), d ** -0.5, dt), _normal(g, (n, I, d), d ** -0.5, dt),
            _normal(g, (n, d, I), I ** -0.5, dt))


def _groups(c, bias):
    """The least popular experts in groups, as the frequency rule forms them: (kept, groups)."""
    order = torch.sort(bias, descending=True, stable=True).indices.tolist()
    K = c["E"] - c["merged"]
    tail = order[K:][::-1]
    return sorted(order[:K]), [tail[i:i + c["group"]] for i in range(0, len(tail), c["group"])]


def _draw_layer(c, seed):
    """The tensors of a layer, from the seed alone."""
    g = _gen(seed)
    dt = DT[c["dtype"]]
    v = {"bias": _bias(c, g), "Wr": _normal(g, (c["E"], c["d"]), c["d"] ** -0.5, dt)}
    kept, groups = _groups(c, v["bias"])
    slot = torch.zeros(c["E"], dtype=torch.int32)
    for j, e in enumerate(kept):
        slot[e] = j
    for j, members in enumerate(groups):
        for e in members:
            slot[e] = len(kept) + j
    v["map"] = slot.to(DEV)
    v["S_r"] = len(kept) + len(groups)
    v["W"] = _experts(c, g, v["S_r"] + c["shared"])
    for b in range(c.get("micro", 1)):
        v["X%d" % b] = _normal(g, (c["T"], c["d"]), 1.0, dt)
        v["dY%d" % b] = _normal(g, (c["T"], c["d"]), 1.0, dt)
    return v


def _prepare_layer(c, seed):
    v = _draw_layer(c, seed)
    T, d, k, I, dt, n_sh, S_r = c["T"], c["d"], c["k"], c["I"], DT[c["dtype"]], c["shared"], v["S_r"]
    S = S_r + n_sh
    R, Rt = T * k, T * (k + n_sh)

    def e(*shape, dtype=dt):
        return torch.empty(shape, dtype=dtype, device=DEV)

    i32, f32, u8 = torch.int32, torch.float32, torch.uint8
    s = dict(c=c, S_r=S_r, map=v["map"], Wr=v["Wr"], bias=v["bias"], W=v["W"])
    s["X"] = [v["X%d" % b] for b in range(c.get("micro", 1))]
    s["dY"] = [v["dY%d" % b] for b in range(c.get("micro", 1))]
    dw = [None] * 3
    if c["kind"] == "train":
        tuning = [j for j in range(S) if j < c["tune"] or j >= S_r]
        s["dW"] = [torch.zeros((len(tuning),) + tuple(w.shape[1:]), dtype=f32, device=DEV) for w in s["W"]]
        dw = [[w[tuning.index(j)] if j in tuning else None for j in range(S)] for w in s["dW"]]
    s["L"] = api.LayerTables(d, I, dt, S_r, n_sh, *[[w[j] for j in range(S)] for w in s["W"]], *dw, device=DEV)
    s.update(idx=e(T, k, dtype=i32), gate=e(T, k, dtype=f32), offsets=e(S_r + 1, dtype=i32),
             perm_token=e(R, dtype=i32), perm_gate=e(R, dtype=f32), inv=e(T, k, dtype=i32), X_perm=e(R, d),
             A_g=e(Rt, I), A_u=e(Rt, I), H=e(Rt, I), O=e(Rt, d), Y=e(T, d),
             ws_perm=e(api.moe_permute_workspace_size(T, k, S_r), dtype=u8),
             ws_fwd=e(api.moe_grouped_swiglu_fwd_workspace_size(s["L"], T, k), dtype=u8))
    if c["kind"] == "train":
        s.update(dO=e(Rt, d), dX_perm=e(Rt, d), dX=e(T, d), dgate=e(T, k, dtype=f32), x_sq=e(T, dtype=f32),
                 dy_sq=e(T, dtype=f32), util=e(S, dtype=f32),
                 ws_bwd=e(api.moe_grouped_swiglu_bwd_workspace_size(s["L"], T, k), dtype=u8))
    return s


def _draw_stack(c, seed):
    g = _gen(seed)
    dt = DT[c["dtype"]]
    layers = []
    for _ in range(c["layers"]):
        lay = dict(bias=_bias(c, g), Wr=_normal(g, (c["E"], c["d"]), c["d"] ** -0.5, dt))
        lay.update(zip(("wg", "wu", "wd"), _experts(c, g, c["E"])))
        if c["shared"]:
            lay.update(zip(("sg", "su", "sd"), _experts(c, g, c["shared"])))
        layers.append(lay)
    return layers, _normal(g, (c["T"], c["d"]), 1.0, dt)


def _draw_merge(c, seed):
    g = _gen(seed)
    dt = DT[c["dtype"]]
    v = {"bias": _bias(c, g), "Wr": _normal(g, (c["E"], c["d"]), c["d"] ** -0.5, dt)}
    v["groups"] = _groups(c, v["bias"])[1]
    v["W"] = _experts(c, g, c["E"])
    v["X"] = _normal(g, (c["T"], c["d"]), 1.0, dt)
    return v


def _prepare_merge(c, seed):
    v = _draw_merge(c, seed)
    E, d, I, dt = c["E"], c["d"], c["I"], DT[c["dtype"]]
    plan = api.plan_from_groups(E, v["groups"])
    G = plan["G"]
    M = [torch.empty((G,) + tuple(w.shape[1:]), dtype=dt, device=DEV) for w in v["W"]]

    def table(mats, n):
        return torch.tensor([m[j].data_ptr() for j in range(n) for m in mats], dtype=torch.int64, device=DEV)

    return dict(c=c, X=v["X"], Wr=v["Wr"], bias=v["bias"], W=v["W"], M=M, G=G, src=table(v["W"], E), dst=table(M, G),
                grp_ptr=torch.from_numpy(plan["grp_ptr"]).to(DEV),
                grp_member=torch.from_numpy(plan["grp_member"]).to(DEV),
                Wq=torch.empty((E, d), dtype=torch.int8, device=DEV), scale=torch.empty(E, device=DEV),
                counts=torch.zeros(E, dtype=torch.int32, device=DEV), alpha=torch.empty(E, device=DEV))


def _prepare_cluster(c, seed):
    """Experts of planted classes (prototype plus noise), counts of a skewed router."""
    g = _gen(seed)
    L, E, d, I, dt = c["layers"], c["E"], c["d"], c["I"], DT[c["dtype"]]
    W = []
    for _ in range(L):
        cls = (torch.randperm(E, generator=g, device=DEV) % c["classes"]).tolist()
        for shape, std in (((I, d), d ** -0.5), ((I, d), d ** -0.5), ((d, I), I ** -0.5)):
            proto = torch.randn((c["classes"],) + shape, generator=g, device=DEV)
            m = torch.empty((E,) + shape, dtype=dt, device=DEV)
            for x in range(E):
                n = torch.randn(shape, generator=g, device=DEV)
                m[x] = n.mul_(0.4 ** 0.5).add_(proto[cls[x]], alpha=0.6 ** 0.5).mul_(std).to(dt)
            W.append(m)
    p = torch.exp(torch.randn((L, E), generator=g, device=DEV))
    counts = (p / p.sum(1, keepdim=True) * 24576).to(torch.int32)
    tuning = torch.zeros((L, E), dtype=torch.uint8, device=DEV)
    tuning.scatter_(1, torch.topk(counts, c["tune"], dim=1).indices, 1)
    src = torch.tensor([W[3 * l + j][x].data_ptr() for l in range(L) for x in range(E) for j in range(3)],
                       dtype=torch.int64, device=DEV)
    return dict(c=c, W=W, src=src, counts=counts, tuning=tuning, B=c["classes"] * L,
                budget=torch.empty(L, dtype=torch.int32, device=DEV),
                labels=torch.empty((L, E), dtype=torch.int32, device=DEV),
                iters=torch.empty(L, dtype=torch.int32, device=DEV),
                ws=torch.empty(api.moe_cluster_workspace_size(L, E, d, I), dtype=torch.uint8, device=DEV))


def prepare(case, seed):
    c = case
    if c["kind"] in ("eval", "train"):
        return _prepare_layer(c, seed)
    if c["kind"] == "merge":
        return _prepare_merge(c, seed)
    if c["kind"] == "cluster":
        return _prepare_cluster(c, seed)
    layers, X = _draw_stack(c, seed)
    return dict(c=c, X=X, stack=QuantizedStack(layers, c["T"], c["k"], device=DEV),
                freq=torch.empty((c["layers"], c["E"]), device=DEV))


# -------------------------------------------------------------------- run ----

def _forward(s, X, x_sq):
    c = s["c"]
    T, k = c["T"], c["k"]
    api.moe_route_topk(X, s["Wr"], s["bias"], k, s["idx"], s["gate"], None)
    api.moe_permute(X, s["idx"], s["gate"], s["map"], s["S_r"], s["offsets"], s["perm_token"], s["perm_gate"],
                    s["inv"], s["X_perm"], s["ws_perm"], E=c["E"], x_sq=x_sq)
    api.moe_grouped_swiglu_fwd(s["L"], X, s["X_perm"], s["offsets"], T, k, s["A_g"], s["A_u"], s["H"], s["O"],
                               s["ws_fwd"])
    api.moe_unpermute(s["L"], s["O"], s["inv"], s["perm_gate"], T, k, s["Y"])


def _backward(s, X, dY, accumulate):
    c = s["c"]
    T, k, gates = c["T"], c["k"], c["gates"]
    api.moe_unpermute_bwd(s["L"], dY, s["O"], s["inv"], s["offsets"], s["perm_gate"], T, k, s["dO"],
                          s["dgate"] if gates else None, dy_sq=s["dy_sq"] if c["utility"] else None)
    api.moe_grouped_swiglu_bwd(s["L"], X, s["X_perm"], s["offsets"], T, k, s["A_g"], s["A_u"], s["H"], s["dO"],
                               s["dX_perm"], accumulate, s["ws_bwd"])
    api.moe_permute_bwd(s["L"], s["dX_perm"], s["inv"], T, k, s["dX"])
    if gates:
        api.moe_route_bwd(s["gate"], s["idx"], s["dgate"], s["Wr"], s["dX"], accumulate=True)


def run(state):
    s, c = state, state["c"]
    if c["kind"] == "eval":
        _forward(s, s["X"][0], None)
        return {"Y": s["Y"], "gate": s["gate"], "idx": s["idx"]}
    if c["kind"] == "train":
        for b in range(c["micro"]):
            _forward(s, s["X"][b], s["x_sq"] if c["utility"] else None)
            _backward(s, s["X"][b], s["dY"][b], b > 0)
        out = {"Y": s["Y"], "dX": s["dX"], "dW_gate": s["dW"][0], "dW_up": s["dW"][1], "dW_down": s["dW"][2]}
        if c["gates"]:
            out["dgate"] = s["dgate"]
        if c["utility"]:
            api.moe_expert_utility(s["L"], s["x_sq"], s["dy_sq"], s["perm_token"], s["perm_gate"], s["offsets"], c["T"],
                                   c["k"], s["ws_bwd"], s["util"])
            out["utility"] = s["util"]
        return out
    if c["kind"] == "profile":
        X = s["stack"].run(s["X"])
        for l in range(c["layers"]):
            api.moe_activation_frequency(s["stack"].counts[l], c["T"], s["freq"][l])
        return {"X": X, "frequency": s["freq"]}
    if c["kind"] == "merge":
        api.moe_quantize_int8(s["Wr"], s["Wq"], s["scale"])
        s["counts"].zero_()
        api.moe_profile_hist(s["X"], s["Wq"], s["scale"], s["bias"], c["k"], s["counts"])
        api.moe_activation_frequency(s["counts"], c["T"], s["alpha"])
        api.moe_merge_experts(s["src"], DT[c["dtype"]], c["d"], c["I"], s["G"], s["grp_ptr"], s["grp_member"],
                              s["alpha"], s["dst"], DT[c["dtype"]])
        return {"frequency": s["alpha"], "M_gate": s["M"][0], "M_up": s["M"][1], "M_down": s["M"][2]}
    api.moe_merge_budget(s["counts"], s["tuning"], 24576, s["B"], s["budget"])
    api.moe_cluster_experts(s["src"], DT[c["dtype"]], c["layers"], c["E"], c["d"], c["I"], s["tuning"], s["budget"],
                            c["r"], 100, s["ws"], s["labels"], None, s["iters"])
    return {"budget": s["budget"], "labels": s["labels"], "iters": s["iters"]}


# ------------------------------------------------------------------- work ----

def work(case):
    """Every input read once, every output written once; the products' flops."""
    c = case
    d, I, E = c["d"], c["I"], c["E"]
    es = 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "cluster":
        n = c["layers"] * (E - c["tune"])
        return {"bytes": n * 3 * d * I * es, "flops": n * (E - c["tune"]) * 3 * d * I}
    T, k = c["T"], c["k"]
    if c["kind"] == "merge":
        g = c["merged"] // c["group"]
        return {"bytes": (c["merged"] + g) * 3 * d * I * es + (T + E) * d * es, "flops": 2 * T * E * d}
    rows = T * (k + c["shared"])
    if c["kind"] == "profile":
        slots = min(E, T * k) + c["shared"]
        return {"bytes": c["layers"] * (slots * 3 * d * I + E * d) + 2 * T * d * es,
                "flops": c["layers"] * (6 * d * I * rows + 2 * T * E * d)}
    S_r = E - c["merged"] + c["merged"] // c["group"]
    slots = min(S_r, T * k) + c["shared"]
    w = {"bytes": slots * 3 * d * I * es + E * d * es + 2 * T * d * es, "flops": 6 * d * I * rows + 2 * T * E * d}
    if c["kind"] == "train":
        # a tuning slot's share of the rows is at least its share of the slots
        tuned = T * (k * c["tune"] // S_r + c["shared"])
        w["bytes"] += (c["tune"] + c["shared"]) * 3 * d * I * 4 + c["micro"] * 2 * T * d * es
        w["flops"] = c["micro"] * (w["flops"] + 6 * d * I * (rows + tuned))
    return w


def tolerance(case):
    c = case
    if c["kind"] == "cluster":
        return {"rel": 0.0, "differ": 0.01}
    if c["kind"] == "merge":
        # one token routed the other way at a near tie moves a frequency by 1 / T
        return {"rel": 1e-5 if c["dtype"] == "f32" else 2e-3, "max": 0.1}
    if c["dtype"] == "f32":
        return {"rel": 1e-4 if c["kind"] == "profile" else 1e-5, "max": 0.01, "differ": 1e-3}
    # bf16 rounding of A, H, O, dA; in a stack also the tokens whose top-k set it changes
    return {"rel": 0.03 if c["kind"] == "profile" else 0.015, "max": 0.99, "differ": 1e-3}


# ------------------------------------------------------------------ exact ----

def _topk64(X, Wr, bias, k):
    logits = X.double() @ Wr.double().t() + bias.double()
    v, idx = torch.sort(logits, dim=1, descending=True, stable=True)
    return idx[:, :k], torch.softmax(v[:, :k], dim=1)


def _swiglu64(x, W):
    wg, wu, wd = (w.double() for w in W)
    ag, au = x @ wg.t(), x @ wu.t()
    s = torch.sigmoid(ag)
    h = ag * s * au
    return ag, au, s, h, h @ wd.t(), (wg, wu, wd)


def _quantised(W):
    """Rows as int8 codes times a scale; the division decides an integer and is defined in fp32."""
    w = W.float().reshape(-1, W.shape[-1])
    s = w.abs().amax(1, keepdim=True) / 127.0
    q = torch.where(s > 0, torch.round(w / s), torch.zeros_like(w)).clamp_(-127, 127)
    return (q.double() * s.double()).reshape(W.shape)


def _exact_layer(c, seed):
    v = _draw_layer(c, seed)
    T, S_r, n_sh = c["T"], v["S_r"], c["shared"]
    train = c["kind"] == "train"
    S = S_r + n_sh
    tuning = [j for j in range(S) if j < c.get("tune", 0) or j >= S_r]
    dW, out = {}, {}
    for b in range(c.get("micro", 1)):
        X, dY = v["X%d" % b].double(), v["dY%d" % b].double()
        idx, gate = _topk64(X, v["Wr"], v["bias"], c["k"])
        slot = v["map"].long()[idx]
        gs = torch.zeros((T, S_r), dtype=torch.float64, device=DEV).scatter_add_(1, slot, gate)
        on = torch.zeros((T, S_r), dtype=torch.bool, device=DEV).scatter_(1, slot, True)
        Y, dX = torch.zeros_like(X), torch.zeros_like(X)
        ds = torch.zeros((T, S_r), dtype=torch.float64, device=DEV)
        util = torch.zeros(S, dtype=torch.float64, device=DEV)
        for j in range(S):
            tok = on[:, j].nonzero()[:, 0] if j < S_r else torch.arange(T, device=DEV)
            if tok.numel() == 0:
                if train and j in tuning and j not in dW:
                    dW[j] = [torch.zeros(w.shape[1:], dtype=torch.float64, device=DEV) for w in v["W"]]
                continue
            g = gs[tok, j, None] if j < S_r else torch.ones((T, 1), dtype=torch.float64, device=DEV)
            x = X[tok]
            ag, au, s, h, o, (wg, wu, wd) = _swiglu64(x, [w[j] for w in v["W"]])
            Y.index_add_(0, tok, g * o)
            if not train:
                continue
            if j < S_r:
                ds[tok, j] = (dY[tok] * o).sum(1)
            do = g * dY[tok]
            dh = do @ wd
            dau = dh * ag * s
            dag = dh * au * s * (1 + ag * (1 - s))
            dX.index_add_(0, tok, dag @ wg + dau @ wu)
            if j in tuning:
                new = [dag.t() @ x, dau.t() @ x, do.t() @ h]
                dW[j] = [p + q for p, q in zip(dW[j], new)] if j in dW else new
            sq = do.square().sum(1) * h.square().sum(1) + (dag.square() + dau.square()).sum(1) * x.square().sum(1)
            util[j] = (tok.numel() * sq.sum()).sqrt()
        out = {"Y": Y, "gate": gate, "idx": idx.int()}
        if train:
            out = {"Y": Y, "dX": dX}
            if c["gates"]:
                out["dgate"] = ds.gather(1, slot)
                dl = gate * (out["dgate"] - (gate * out["dgate"]).sum(1, keepdim=True))
                dense = torch.zeros((T, c["E"]), dtype=torch.float64, device=DEV).scatter_(1, idx, dl)
                dX += dense @ v["Wr"].double()
            if c["utility"]:
                out["utility"] = util
    if train:
        for i, name in enumerate(("dW_gate", "dW_up", "dW_down")):
            out[name] = torch.stack([dW[j][i] for j in tuning])
    return out


def _exact_stack(c, seed):
    layers, X = _draw_stack(c, seed)
    X = X.double()
    freq = torch.zeros((c["layers"], c["E"]), dtype=torch.float64, device=DEV)
    for l, lay in enumerate(layers):
        Xn = X / torch.sqrt(X.square().mean(1, keepdim=True) + 1e-6)
        idx, gate = _topk64(Xn, _quantised(lay["Wr"]), lay["bias"], c["k"])
        freq[l] = torch.bincount(idx.reshape(-1), minlength=c["E"]).double() / c["T"]
        Y = torch.zeros_like(X)
        for e in range(c["E"]):
            tok, j = (idx == e).nonzero(as_tuple=True)
            if tok.numel():
                o = _swiglu64(Xn[tok], [_quantised(lay[n][e]) for n in ("wg", "wu", "wd")])[4]
                Y.index_add_(0, tok, gate[tok, j, None] * o)
        for i in range(c["shared"]):
            Y += _swiglu64(Xn, [_quantised(lay[n][i]) for n in ("sg", "su", "sd")])[4]
        X = X + Y
    return {"X": X, "frequency": freq}


def _exact_merge(c, seed):
    v = _draw_merge(c, seed)
    idx, _ = _topk64(v["X"], _quantised(v["Wr"]), v["bias"], c["k"])
    f = torch.bincount(idx.reshape(-1), minlength=c["E"]).double() / c["T"]
    out = {"frequency": f}
    for name, W in zip(("M_gate", "M_up", "M_down"), v["W"]):
        M = torch.empty((len(v["groups"]),) + tuple(W.shape[1:]), dtype=torch.float64, device=DEV)
        for j, members in enumerate(v["groups"]):
            a = f[members]
            a = a / a.sum() if float(a.sum()) > 0 else torch.full_like(a, 1.0 / len(members))
            M[j] = sum(a[i] * W[e].double() for i, e in enumerate(members))
        out[name] = M
    return out


def exact(case, seed):
    c = case
    if c["kind"] in ("eval", "train"):
        return _exact_layer(c, seed)
    if c["kind"] == "profile":
        return _exact_stack(c, seed)
    if c["kind"] == "merge":
        return _exact_merge(c, seed)
    return None   # whole numbers only
