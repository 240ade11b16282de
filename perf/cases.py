"""The calls that programs make of this library, as measurable cases.

The library is one MoE expert layer: a forward and a chunked-recompute
backward over token-slots grouped by expert, the planner that chooses the
chunk count from an activation budget, and the router in front of the layer.
So there are four kinds of case, each one pass of a program's loop:

* ``serve``   the allocation-free forward of a serving loop, a few tokens at
              a time; every local expert's weights are read for a handful of
              rows each.
* ``forward`` the forward alone (prefill, evaluation): hundreds to thousands
              of tokens.
* ``step``    one training step of the layer: expert counts, the plan for the
              activation budget, forward, backward; with ``micro`` > 1 the
              weight gradients of several micro-batches are accumulated;
              ``order`` selects the chunk order.
* ``router``  router forward and backward on a batch of tokens.
* ``block``   the trainable block, router -> layer -> layer backward ->
              router backward adding into the layer's input gradient.

Sizes are those of the seeded workloads in moe_workloads.py, of the tests, or
generic ones of the same ranges.  Routing is skewed as a trained router's is:
expert loads from a Dirichlet or Zipf law, or one hot expert.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2511_21431_amd as mf

BINS = (1, 2, 4, 8, 16)


def listed():
    return [
        # A serving loop's decode step: 16 sequences, 32 fine-grained local experts.
        dict(name="serve_decode_16", kind="serve", dtype="bf16", T=16, h=7168, F=2048, E=32, k=8,
             loads="dirichlet", skew=5.0),
        # Prefill of about a thousand tokens through many small experts.
        dict(name="forward_prefill_1000", kind="forward", dtype="bf16", T=1000, h=2048, F=1408,
             E=64, k=6, loads="dirichlet", skew=2.0, chunks=1),
        # The smallest training call (workload 1): fp32, launch latency.
        dict(name="step_tiny_f32", kind="step", dtype="f32", T=256, h=64, F=128, E=4, k=2,
             loads="dirichlet", skew=5.0, budget=1 << 30, micro=1, order="tokens"),
        # fp32 training of an ordinary small layer (reference runs, debugging of numerics).
        dict(name="step_f32", kind="step", dtype="f32", T=2048, h=1024, F=1408, E=8, k=2,
             loads="dirichlet", skew=5.0, budget=1 << 30, micro=1, order="tokens"),
        # Workload 2: balanced experts, two chunks.
        dict(name="step_balanced", kind="step", dtype="bf16", T=8192, h=2048, F=1408, E=16, k=4,
             loads="dirichlet", skew=5.0, budget=250_000_000, micro=1, order="tokens"),
        # Ragged sizes (T prime, F and h off the tile sizes), gradient accumulation over
        # two micro-batches.
        dict(name="step_ragged_accumulate", kind="step", dtype="bf16", T=3001, h=1600, F=960, E=20,
             k=5, loads="dirichlet", skew=1.0, budget=100_000_000, micro=2, order="tokens"),
        # Workload 3: few large experts with a dense-size FFN, Zipf loads, eight chunks.
        dict(name="step_dense_ffn", kind="step", dtype="bf16", T=16384, h=4096, F=14336, E=8, k=2,
             loads="zipf", skew=1.2, budget=500_000_000, micro=1, order="tokens"),
        # Workload 4: fine-grained experts, one at 8 times the mean load, four chunks.
        dict(name="step_fine_grained", kind="step", dtype="bf16", T=8192, h=7168, F=2048, E=32,
             k=8, loads="hot", skew=0.25, budget=1_000_000_000, micro=1, order="tokens"),
        # The same step with expert-ordered chunks.
        dict(name="step_expert_order", kind="step", dtype="bf16", T=8192, h=7168, F=2048, E=32,
             k=8, loads="hot", skew=0.25, budget=1_000_000_000, micro=1, order="experts"),
        # Workload 5, the benchmark's step: the per-GPU worst case, half of all slots on one
        # expert, eight chunks.
        dict(name="step_worst_case", kind="step", dtype="bf16", T=131072, h=7168, F=2048, E=32,
             k=8, loads="hot", skew=0.5, budget=8_000_000_000, micro=1, order="tokens"),
        # The router of a 256-expert model.
        dict(name="router_256", kind="router", dtype="bf16", T=32768, h=7168, E=256, k=8),
        # Router and layer trained together, 64 experts.
        dict(name="block_64", kind="block", dtype="bf16", T=4096, h=2048, F=704, E=64, k=6,
             chunks=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _log_64(rng, lo, hi):
    return max(lo, _log_int(rng, lo, hi) // 64 * 64)


def _loads(rng):
    kind = rng.choice(("dirichlet", "dirichlet", "zipf", "hot"))
    skew = {"dirichlet": rng.uniform(0.7, 6.0), "zipf": rng.uniform(0.6, 1.4),
            "hot": rng.uniform(0.1, 0.5)}[kind]
    return kind, round(skew, 3)


def draw(rng):
    most_flops, most_bytes = 3.4e14, 6e9
    kind = rng.choice(("serve", "forward", "step", "step", "step", "router", "block"))
    if kind == "router":
        while True:
            c = dict(kind=kind, dtype="f32" if rng.random() < 0.2 else "bf16",
                     T=_log_int(rng, 300, 131072), h=_log_64(rng, 512, 7168),
                     E=rng.choice((rng.randint(8, 256), 8, 16, 32, 64, 128, 160, 256)))
            c["k"] = rng.randint(2, min(8, c["E"]))  # (one slot: its gate is 1, no gradient)
            if c["T"] * c["h"] * (2 if c["dtype"] == "bf16" else 4) < 2e9:
                return c
    if kind == "block":
        while True:
            E = rng.choice((8, 16, 32, 64, 64, 128))
            c = dict(kind=kind, dtype="bf16", T=_log_int(rng, 500, 8192),
                     h=_log_64(rng, 512, 4096), F=_log_64(rng, 256, 2048), E=E,
                     k=rng.randint(2, 8), chunks=rng.choice((1, 1, 2)))
            if 3 * E * c["h"] * c["F"] * 4 <= most_bytes:
                return c
    while True:
        c = dict(kind=kind, dtype="bf16")
        f32 = kind == "step" and rng.random() < 0.25
        if f32:
            c.update(dtype="f32", T=_log_int(rng, 64, 8192), h=_log_64(rng, 64, 2048),
                     F=_log_64(rng, 64, 2816), E=rng.randint(2, 16))
        elif kind == "serve":
            c.update(T=_log_int(rng, 1, 128), h=_log_64(rng, 1024, 7168),
                     F=_log_64(rng, 512, 4096), E=rng.choice((8, 16, 20, 32, 64)))
        elif kind == "forward":
            c.update(T=_log_int(rng, 200, 16384), h=_log_64(rng, 512, 7168),
                     F=_log_64(rng, 512, 8192), E=rng.choice((4, 8, 13, 16, 32, 64)))
        else:
            c.update(T=_log_int(rng, 500, 65536), h=_log_64(rng, 512, 7168),
                     F=_log_64(rng, 512, 14336), E=rng.choice((4, 8, 12, 16, 20, 32, 64)))
        c["k"] = rng.randint(1, min(8, c["E"]))
        c["loads"], c["skew"] = _loads(rng)
        es = 4 if f32 else 2
        N, hF = c["T"] * c["k"], c["h"] * c["F"]
        if 22 * N * hF > (1e12 if f32 else most_flops) or 12 * c["E"] * hF > most_bytes:
            continue
        if c["T"] * c["h"] * es >= 1 << 31 or 2 * hF * es >= 1 << 31:
            continue
        if kind == "serve":
            return c
        if kind == "forward":
            c["chunks"] = rng.choice((1, 1, 2, 4))
            return c
        need = N * max(es * (2 * c["h"] + 2 * c["F"]), es * (3 * c["F"] + c["h"]) + c["F"] // 8)
        c["budget"] = int(need / rng.choice((0.5, 0.9, 1.6, 3.0, 6.0))) + (1 << 20)
        c["micro"] = rng.choice((1, 1, 1, 2))
        c["order"] = rng.choice(("tokens", "tokens", "tokens", "experts"))
        return c


# ---------------------------------------------------------------- inputs
def _routing(c, seed, n):
    """idx [T, k] with the loads of the case, gates softmax over the slots."""
    rng = np.random.default_rng([int(seed), 7, n])
    T, E, k = c["T"], c["E"], c["k"]
    if c["loads"] == "dirichlet":
        p = rng.dirichlet(np.full(E, c["skew"]))
    elif c["loads"] == "zipf":
        p = np.empty(E)
        p[rng.permutation(E)] = np.arange(1, E + 1, dtype=np.float64) ** -c["skew"]
        p /= p.sum()
    else:
        p = np.empty(E)
        hot = int(rng.integers(E))
        p[np.arange(E) != hot] = rng.dirichlet(np.ones(E - 1)) * (1 - c["skew"]) if E > 1 else 0
        p[hot] = c["skew"] if E > 1 else 1.0
    raw = p * (T * k)
    counts = np.floor(raw).astype(np.int64)
    counts[np.argsort(counts - raw, kind="stable")[:T * k - int(counts.sum())]] += 1
    idx = np.repeat(np.arange(E, dtype=np.int32), counts)
    rng.shuffle(idx)
    g = rng.standard_normal((T, k))
    g = np.exp(g - g.max(1, keepdims=True))
    g /= g.sum(1, keepdims=True)
    return (torch.from_numpy(idx.reshape(T, k)).cuda(),
            torch.from_numpy(g.astype(np.float32)).cuda())


def _normal(gen, shape, std, dtype):
    t = torch.empty(shape, dtype=dtype, device="cuda")
    flat = t.view(-1)
    for i in range(0, flat.numel(), 1 << 27):
        j = min(flat.numel(), i + (1 << 27))
        flat[i:j] = torch.randn(j - i, generator=gen, device="cuda").mul_(std)
    return t


def _inputs(c, seed):
    """Everything that comes from the seed: a dict of tensors; the per-micro-batch
    ones in lists."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 1000003 + 29)
    bf16 = c["dtype"] == "bf16"
    dt = torch.bfloat16 if bf16 else torch.float32
    T, h, E, k = c["T"], c["h"], c["E"], c["k"]
    s = {}
    if c["kind"] in ("router", "block"):
        s["Wr"] = _normal(gen, (E, h), h ** -0.5, dt)
    if c["kind"] == "router":
        s["X"] = _normal(gen, (T, h), 1.0, dt)
        # what a forward pass saved and the layer's backward gave
        z = torch.randn((T, E), generator=gen, device="cuda")
        top, idx = z.topk(k, dim=1)
        s["idx"], s["gates"] = idx.int().contiguous(), torch.softmax(top, 1).contiguous()
        s["dgates"] = torch.randn((T, k), generator=gen, device="cuda")
        return s
    F, n = c["F"], c.get("micro", 1)
    s["W1"] = _normal(gen, (E, 2 * F, h), 0.02 if bf16 else h ** -0.5, dt)
    s["W2"] = _normal(gen, (E, h, F), 0.02 if bf16 else F ** -0.5, dt)
    s["X"] = [_normal(gen, (T, h), 1.0, dt) for _ in range(n)]
    if c["kind"] in ("step", "block"):
        s["dY"] = [_normal(gen, (T, h), 1.0, dt) for _ in range(n)]
    if c["kind"] != "block":
        r = [_routing(c, seed, i) for i in range(n)]
        s["idx"], s["gates"] = [x[0] for x in r], [x[1] for x in r]
    return s


def prepare(case, seed):
    c = case
    T, h, E, k, F = c["T"], c["h"], c["E"], c["k"], c.get("F", 64)
    bf16 = c["dtype"] == "bf16"
    dt = torch.bfloat16 if bf16 else torch.float32
    s = _inputs(c, seed)
    s["case"] = c
    s["shape"] = mf.make_shape(T, h, F, E, k, mf.BF16 if bf16 else mf.F32)
    new = lambda *shape, dtype=dt: torch.empty(shape, dtype=dtype, device="cuda")  # noqa: E731
    f32, i32 = torch.float32, torch.int32
    n = c.get("micro", 1)
    if c["kind"] in ("router", "block"):
        s.update(r_idx=new(T, k, dtype=i32), r_gates=new(T, k, dtype=f32),
                 r_logits=new(T, E, dtype=f32), dWr=new(E, h, dtype=f32))
    if c["kind"] == "router":
        s["dX"] = new(T, h)
        return s
    s["Y"] = [new(T, h) for _ in range(n)]
    if c["kind"] in ("step", "block"):
        s.update(dX=[new(T, h) for _ in range(n)], dg=[new(T, k, dtype=f32) for _ in range(n)],
                 dW1=new(E, 2 * F, h, dtype=f32), dW2=new(E, h, F, dtype=f32),
                 work=new(E + 1, dtype=i32))
    return s


# ------------------------------------------------------------------ passes
def _step(s, c):
    sh = s["shape"]
    for i in range(c["micro"]):
        x, idx, g = s["X"][i], s["idx"][i], s["gates"][i]
        counts = mf.memfine_count(sh, idx, s["work"])
        _, C, _ = mf.memfine_plan(sh, counts, c["budget"], bins=BINS)
        mf.memfine_moe_fwd(sh, C, x, idx, g, s["W1"], s["W2"], s["Y"][i])
        mf.memfine_moe_bwd(sh, C, x, idx, g, s["W1"], s["W2"], s["dY"][i], s["dX"][i], s["dW1"],
                           s["dW2"], s["dg"][i], accumulate_dW=i > 0)
    return {"Y": s["Y"], "dX": s["dX"], "dgates": s["dg"], "dW1": s["dW1"], "dW2": s["dW2"]}


def run(state):
    s, c = state, state["case"]
    sh = s["shape"]
    if c["kind"] == "serve":
        mf.memfine_moe_fwd_noalloc(sh, 1, s["X"][0], s["idx"][0], s["gates"][0], s["W1"], s["W2"],
                                   s["Y"][0])
        return s["Y"][0]
    if c["kind"] == "forward":
        mf.memfine_moe_fwd(sh, c["chunks"], s["X"][0], s["idx"][0], s["gates"][0], s["W1"],
                           s["W2"], s["Y"][0])
        return s["Y"][0]
    if c["kind"] == "step":
        if c["order"] == "tokens":
            return _step(s, c)
        mf.memfine_set_launch_options(chunk_order=mf.CHUNK_EXPERTS)
        try:
            return _step(s, c)
        finally:
            mf.memfine_set_launch_options()
    if c["kind"] == "router":
        mf.memfine_router_fwd(sh, s["X"], s["Wr"], s["r_idx"], s["r_gates"], s["r_logits"])
        mf.memfine_router_bwd(sh, s["X"], s["Wr"], s["idx"], s["gates"], s["dgates"], s["dX"],
                              s["dWr"])
        return {"idx": s["r_idx"], "gates": s["r_gates"], "logits": s["r_logits"], "dX": s["dX"],
                "dWr": s["dWr"]}
    x, idx, g, C = s["X"][0], s["r_idx"], s["r_gates"], c["chunks"]
    mf.memfine_router_fwd(sh, x, s["Wr"], idx, g, s["r_logits"])
    mf.memfine_moe_fwd(sh, C, x, idx, g, s["W1"], s["W2"], s["Y"][0])
    mf.memfine_moe_bwd(sh, C, x, idx, g, s["W1"], s["W2"], s["dY"][0], s["dX"][0], s["dW1"],
                       s["dW2"], s["dg"][0])
    mf.memfine_router_bwd(sh, x, s["Wr"], idx, g, s["dg"][0], s["dX"][0], s["dWr"],
                          accumulate_dX=True)
    return {"idx": idx, "gates": g, "logits": s["r_logits"], "Y": s["Y"][0], "dX": s["dX"][0],
            "dW1": s["dW1"], "dW2": s["dW2"], "dWr": s["dWr"]}


def work(case):
    """Flops that the results need (the backward's recomputation of FC1 is part of
    the method) and each input read, each output written once."""
    c = case
    T, h, E, k, F = c["T"], c["h"], c["E"], c["k"], c.get("F", 0)
    es = 2 if c["dtype"] == "bf16" else 4
    N, hF, n = T * k, h * F, c.get("micro", 1)
    flops = bytes_ = 0.0
    if c["kind"] in ("serve", "forward"):
        e_hit = min(E, N)
        return {"flops": 6.0 * N * hF, "bytes": es * (2.0 * T * h + 3.0 * e_hit * hF) + 8.0 * N}
    if c["kind"] in ("step", "block"):
        flops += n * 22.0 * N * hF
        bytes_ += n * (es * 4.0 * T * h + 12.0 * N) + es * 3.0 * E * hF + 4.0 * 3.0 * E * hF
    if c["kind"] in ("router", "block"):
        flops += 6.0 * T * E * h
        bytes_ += es * (2.0 * T * h + E * h) + 4.0 * E * h + 4.0 * T * E + 20.0 * N
    return {"flops": flops, "bytes": bytes_}


def tolerance(case):
    # About four times the error measured against exact(): at most 1.3e-6 on the fp32 path
    # (dX of step_f32; 3.5e-7 on the tiny step), 3.0e-3 to 3.7e-3 for Y and dX with bf16
    # inputs, intermediates and results.  `differ`: router ids of logits equal to fp32 rounding.
    if case["dtype"] == "f32":
        return {"rel": 6e-6, "differ": 1e-3}
    return {"rel": 1.3e-2, "differ": 1e-3}


# ------------------------------------------------------- 64-bit reference
def _layer64(c, x, idx, gates, W1, W2, dY, dW1, dW2):
    """Y, and with dY the gradients, expert by expert in float64; dW1 and dW2 are
    added to."""
    T, h, E, F = c["T"], c["h"], c["E"], c["F"]
    f64 = dict(dtype=torch.float64, device="cuda")
    Y = torch.zeros((T, h), **f64)
    dX = torch.zeros((T, h), **f64) if dY is not None else None
    dg = torch.zeros(idx.numel(), **f64) if dY is not None else None
    flat = idx.reshape(-1).long()
    for e in range(E):
        slots = (flat == e).nonzero()[:, 0]
        if slots.numel() == 0:
            continue
        w1, w2 = W1[e].double(), W2[e].double()
        for part in slots.split(32768):
            tok = part // c["k"]
            g = gates.reshape(-1)[part].double()[:, None]
            xe = x[tok].double()
            u = xe @ w1.T
            ug, uu = u[:, :F], u[:, F:]
            s = torch.sigmoid(ug)
            act = ug * s * uu
            Y.index_add_(0, tok, g * (act @ w2.T))
            if dY is None:
                continue
            dy = dY[tok].double()
            dA = dy @ w2
            dg[part] = (dA * act).sum(1)
            da = g * dA
            du = torch.cat((da * uu * s * (1 + ug * (1 - s)), da * ug * s), 1)
            dX.index_add_(0, tok, du @ w1)
            dW2[e] += dy.T @ (g * act)
            dW1[e] += du.T @ xe
    return Y, dX, None if dg is None else dg.reshape(idx.shape)


def exact(case, seed):
    c, s = case, _inputs(case, seed)
    f64 = dict(dtype=torch.float64, device="cuda")
    T, h, E, k, F = c["T"], c["h"], c["E"], c["k"], c.get("F", 0)

    def router_fwd(x):
        logits = torch.empty((T, E), **f64)
        for t in range(0, T, 16384):
            logits[t:t + 16384] = x[t:t + 16384].double() @ s["Wr"].double().T
        top, idx = logits.topk(k, dim=1)
        return logits, idx.int(), torch.softmax(top, 1)

    def router_bwd(x, idx, gates, dg, dX):
        g = gates.double()
        dz = g * (dg.double() - (g * dg.double()).sum(1, keepdim=True))
        D = torch.zeros((T, E), **f64).scatter_add_(1, idx.long(), dz)
        dWr = torch.zeros((E, h), **f64)
        for t in range(0, T, 16384):
            dX[t:t + 16384] += D[t:t + 16384] @ s["Wr"].double()
            dWr += D[t:t + 16384].T @ x[t:t + 16384].double()
        return dWr

    if c["kind"] in ("serve", "forward"):
        return _layer64(c, s["X"][0], s["idx"][0], s["gates"][0], s["W1"], s["W2"], None, None,
                        None)[0]
    if c["kind"] == "router":
        logits, _, gates = router_fwd(s["X"])
        dX = torch.zeros((T, h), **f64)
        dWr = router_bwd(s["X"], s["idx"], s["gates"], s["dgates"], dX)
        return {"idx": None, "gates": gates, "logits": logits, "dX": dX, "dWr": dWr}
    dW1, dW2 = torch.zeros((E, 2 * F, h), **f64), torch.zeros((E, h, F), **f64)
    if c["kind"] == "step":
        out = {"Y": [], "dX": [], "dgates": [], "dW1": dW1, "dW2": dW2}
        for i in range(c["micro"]):
            r = _layer64(c, s["X"][i], s["idx"][i], s["gates"][i], s["W1"], s["W2"], s["dY"][i],
                         dW1, dW2)
            for name, v in zip(("Y", "dX", "dgates"), r):
                out[name].append(v)
        return out
    logits, idx, gates = router_fwd(s["X"][0])
    Y, dX, dg = _layer64(c, s["X"][0], idx, gates, s["W1"], s["W2"], s["dY"][0], dW1, dW2)
    dWr = router_bwd(s["X"][0], idx, gates, dg, dX)
    return {"idx": None, "gates": gates, "logits": logits, "Y": Y, "dX": dX, "dW1": dW1,
            "dW2": dW2, "dWr": dWr}
