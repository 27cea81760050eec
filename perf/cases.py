"""The work whose speed counts: MoE-layer passes as a serving program makes them, through the package's public calls.

A case is a dict of plain values.  Fields of every case:
  api    "layer"   MoELayer.forward on resident hidden states (router, rerouting, experts, combine)
         "stack"   MoEStack.forward, the pre-norm residual chain of layers
         "calls"   the same layer pass as separate calls of the package's functions, outputs allocated by them
         "permute" moe_reroute_permute alone, on given expert ids
  T      tokens of the batch
  M, k   routed experts and experts per token
  N, aid adapters in the pool (16 slots each), and how the tokens' adapters are drawn: "uniform" over base and adapters,
         "zipf" (1.1), "power" (adapters only, power-law shape 0.3), "base" (no adapter traffic)
Layers also have H, I, S (shared experts), dtype, renorm, bias (added to the gate logits of the experts that the token's
adapter tuned), lo / hi (experts an adapter tunes) and, for stacks, L layers.
"""
import math

import numpy as np
import torch

import paper_2508_17624_amd as ew
from paper_2508_17624_amd.layer import MoELayer, MoEStack, load_layer

SLOTS_PER_ADAPTER = 16
# The layer of configurations 1, 2 and 4 (hidden 2048, 64 experts of 1408, two shared experts, top-6).
BASE = dict(H=2048, I=1408, M=64, k=6, S=2, dtype="bf16", renorm=False, bias=0.0, lo=2, hi=16)


def _layer(name, T, N, aid, **kw):
    return dict(dict(BASE, api="layer", T=T, N=N, aid=aid, L=1, name=name), **kw)


def listed():
    return [
        # configuration 0: a layer so small that only calls and launches count; fp32, as a user checks a port against a reference
        _layer("tiny_f32", 64, 2, "uniform", H=256, I=128, M=8, k=2, S=1, dtype="f32", lo=2, hi=2),
        # one user's next token: the least work a decode step can have
        _layer("decode_1", 1, 4, "uniform", lo=6, hi=6),
        # a few users on many adapters: ragged batch, another layer shape, renormalised top-4 weights
        _layer("decode_13", 13, 20, "uniform", H=1024, I=896, M=96, k=4, S=1, renorm=True),
        # configuration 1: the ordinary decode batch
        _layer("decode_64", 64, 4, "uniform", lo=6, hi=6),
        # a program that does its own buffering and calls the operations one by one; no shared experts
        _layer("calls_48", 48, 8, "zipf", api="calls", H=1536, I=768, M=64, k=4, S=0),
        # four of configuration 4's 26 layers: a full decode batch over 20 adapters
        _layer("stack_256", 256, 20, "uniform", api="stack", L=4),
        # a chunk of a chunked prefill: skewed popularity, specialised adapters, no base traffic
        _layer("chunk_512", 512, 20, "power", bias=2.0),
        # a ragged prompt batch on a layer of many small experts without shared ones
        _layer("prefill_1999", 1999, 10, "zipf", H=1536, I=640, M=128, k=8, S=0),
        # configuration 2's prefill with base-model traffic only, what the 20-adapter figure is compared with
        _layer("prefill_8192_base", 8192, 20, "base", bias=2.0),
        # configuration 2: the headline prefill
        _layer("prefill_8192", 8192, 20, "zipf", bias=2.0),
        # dispatch bookkeeping alone, for experts that run elsewhere: a ragged batch, and configuration 3
        dict(api="permute", name="permute_30011", T=30011, M=128, k=8, N=7, aid="zipf", lo=2, hi=16),
        dict(api="permute", name="permute_1M", T=1 << 20, M=64, k=6, N=20, aid="uniform", lo=2, hi=16),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    api = rng.choice(["layer", "layer", "layer", "layer", "calls", "stack", "permute", "f32"])
    aid = rng.choice(["uniform", "zipf", "power", "base"])
    lo = rng.randint(2, 8)
    if api == "permute":
        return dict(api=api, T=_log_int(rng, 4096, 1 << 20), M=rng.choice([64, 96, 128]), k=rng.choice([2, 4, 6]), N=rng.randint(1, 20),
                    aid=aid, lo=lo, hi=16)
    if api == "f32":
        return dict(api="layer", T=_log_int(rng, 1, 256), H=64 * rng.randint(2, 6), I=32 * rng.randint(2, 8), M=rng.choice([8, 12, 16]), k=2,
                    S=rng.randint(0, 2), N=rng.randint(1, 4), aid=aid, L=1, dtype="f32", renorm=rng.random() < 0.5, bias=0.0, lo=1, hi=4)
    H, I = rng.choice([(2048, 1408), (1024, 896), (1536, 768), (1536, 640), (1280, 512), (2048, 1024)])
    c = dict(api=api, H=H, I=I, M=rng.choice([48, 64, 96]), k=rng.choice([2, 4, 6, 8]), S=rng.randint(0, 2), N=rng.randint(1, 20), aid=aid,
             L=1, dtype="bf16", renorm=rng.random() < 0.3, bias=rng.choice([0.0, 2.0]), lo=lo, hi=16)
    if api == "stack":
        return dict(c, L=rng.randint(2, 3), T=_log_int(rng, 1, 256), bias=0.0, M=64, renorm=False)
    if api == "calls":
        return dict(c, T=_log_int(rng, 1, 512))
    return dict(c, T=_log_int(rng, 1, 4096 if c["k"] + c["S"] > 8 else 8192))


# ------------------------------------------------------------------------------------------------ inputs
def _tuned(c, rs):
    """Ascending ids of the experts each adapter tunes."""
    return [np.sort(rs.choice(c["M"], size=int(rs.integers(c["lo"], c["hi"] + 1)), replace=False)).astype(np.int32) for _ in range(c["N"])]


def _class_shares(c):
    """Share of the tokens of each class: base, adapter 1, ... N."""
    N = c["N"]
    if c["aid"] == "base":
        p = np.eye(1, N + 1)[0]
    elif c["aid"] == "uniform":
        p = np.ones(N + 1)
    elif c["aid"] == "zipf":
        p = np.arange(1, N + 2) ** -1.1
    else:  # x in (0, 1] with density a x^(a-1), adapter 1 + floor(N x)
        edge = (np.arange(N + 1) / N) ** 0.3
        p = np.concatenate([[0.0], np.diff(edge)])
    return p / p.sum()


def _aid(c, rs):
    return torch.from_numpy(rs.choice(c["N"] + 1, size=c["T"], p=_class_shares(c)).astype(np.int32)).cuda()


def prepare(case, seed):
    c = case
    rs = np.random.default_rng([seed, c["T"], c["M"]])
    g = torch.Generator(device="cuda").manual_seed(int(rs.integers(1 << 40)))
    P = c["M"] + c["N"] * SLOTS_PER_ADAPTER
    if c["api"] == "permute":
        emap = np.tile(np.arange(c["M"], dtype=np.int32), (c["N"] + 1, 1))
        for a, ids in enumerate(_tuned(c, rs), start=1):
            emap[a, ids] = c["M"] + (a - 1) * SLOTS_PER_ADAPTER + np.arange(len(ids))
        ids = torch.rand((c["T"], c["M"]), generator=g, device="cuda").topk(c["k"], dim=1).indices.to(torch.int32)
        return dict(case=c, ids=ids.contiguous(), aid=_aid(c, rs), emap=torch.from_numpy(emap).cuda(), P=P)
    H, I, M, S, L = c["H"], c["I"], c["M"], c["S"], c["L"]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    el = 2 if c["dtype"] == "bf16" else 4

    def normal(*shape, std=0.02, dtype=dt):
        return torch.randn(shape, generator=g, device="cuda", dtype=dtype).mul_(std)

    # the pool as a server has it: pages under the loaded experts only; a stack's in larger pages, as its number of layers asks for
    pool = ew.ExpertPool(L, M, c["N"], SLOTS_PER_ADAPTER, 2 * I * H * el, H * I * el, page_bytes=(8 << 20) if L > 1 else 0)
    gates, shared, bias = [], [], None
    for layer in range(L):
        tuned = _tuned(c, rs)
        load_layer(pool, layer, (normal(M, 2 * I, H), normal(M, H, I)), [(normal(len(t), 2 * I, H), normal(len(t), H, I)) for t in tuned], tuned)
        gates.append(normal(M, H, dtype=torch.float32))
        shared.append((normal(S, 2 * I, H), normal(S, H, I)) if S else (None, None))
        if c["bias"]:
            bias = torch.zeros((c["N"] + 1, M), dtype=torch.float32)
            for a, ids in enumerate(tuned, start=1):
                bias[a, torch.from_numpy(ids).long()] = c["bias"]
            bias = bias.cuda()
    st = dict(case=c, pool=pool, x=normal(c["T"], H, std=1.0), aid=_aid(c, rs), P=P)
    if c["api"] == "stack":
        st["stack"] = MoEStack(pool, gates, shared, c["k"], I, c["T"], dt)
    elif c["api"] == "layer":
        st["layer"] = MoELayer(pool, 0, gates[0], shared[0][0], shared[0][1], c["k"], I, c["T"], dt, bias=bias, renormalize=c["renorm"])
    else:
        st.update(Wg=gates[0], shared=shared[0], bias=bias, view=pool.view(0), emap=pool.expert_map_host(0).cuda())
    return st


# ------------------------------------------------------------------------------------------------ one pass
def run(state):
    c = state["case"]
    if c["api"] == "permute":
        slot, counts, offsets, pair_of_row, row_of_pair = ew.moe_reroute_permute(state["ids"], state["aid"], state["emap"], c["N"], state["P"])
        return dict(slot=slot, counts=counts, offsets=offsets, pair_of_row=pair_of_row, row_of_pair=row_of_pair)
    x, aid = state["x"], state["aid"]
    if c["api"] == "stack":
        return state["stack"].forward(x, aid)
    if c["api"] == "layer":
        layer = state["layer"]
        out = layer.forward(x, aid)
        return dict(out=out, ids=layer.ids, w=layer.w)
    T, k, P = c["T"], c["k"], state["P"]
    w13, w2, _, _ = state["view"]
    logits = ew.moe_gate_logits(x, state["Wg"], aid if state["bias"] is not None else None, state["bias"])
    ids, w, _, counts, offsets, por, rop = ew.moe_route_reroute_permute(logits, aid, state["emap"], k, c["N"], P, renormalize=c["renorm"])
    if c["S"]:
        y = ew.moe_grouped_ffn_with_shared(x, k, c["I"], P, counts, offsets, por, w13, w2, *state["shared"])
        out = ew.moe_unpermute(y, rop, w, shared_out=y[T * k:])
    else:
        y = ew.moe_grouped_ffn(x, k, c["I"], P, counts, offsets, por, w13, w2)
        out = ew.moe_unpermute(y, rop, w)
    return dict(out=out, ids=ids, w=w)


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def _active(c):
    """Expected number of routed slots that at least one token visits, for a router that spreads its tokens evenly."""
    p, hit, M = _class_shares(c), c["k"] / c["M"], c["M"]
    tuned = (c["lo"] + c["hi"]) / 2 / M
    lift = 1.0
    if c.get("bias"):   # +2.0 on a logit of spread about 1: a tuned expert is picked about five times as often as another one
        lift = 5.0 / (tuned * 5.0 + 1 - tuned)
    n = sum(tuned * M * (1 - (1 - q * min(1.0, hit * lift)) ** c["T"]) for q in p[1:])
    base = sum(q * (1 if a == 0 else 1 - tuned) for a, q in enumerate(p))
    return n + M * (1 - (1 - base * hit) ** c["T"])


def work(case):
    c = case
    T, M, k = c["T"], c["M"], c["k"]
    P = M + c["N"] * SLOTS_PER_ADAPTER
    if c["api"] == "permute":
        return {"bytes": T * (4 * k + 4) + 3 * T * k * 4 + 4 * (2 * P + 1) + 4 * (c["N"] + 1) * M, "flops": 0}
    H, I, S, L = c["H"], c["I"], c["S"], c["L"]
    el = 2 if c["dtype"] == "bf16" else 4
    weights = (_active(c) + S) * 3 * H * I * el
    per_layer = weights + M * H * 4 + 2 * T * H * el + 4 * T * (1 + 2 * k)
    flops = T * (k + S) * 6 * H * I + 2 * T * H * M
    return {"bytes": L * per_layer, "flops": L * flops}


def tolerance(case):
    if case["api"] == "permute":
        return "exact"
    # router scores are fp32 sums: two near-equal experts may change places ("differ"), which moves that token's output ("max")
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}
    return {"rel": 1e-2, "max": 0.3, "differ": 1e-3}
