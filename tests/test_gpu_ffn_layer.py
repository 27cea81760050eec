"""GPU parity: grouped SwiGLU FFN, un-permute, gate logits and the whole layer, against the fp64
oracle.  bf16 tolerance (stated by the benchmark spec): relative L2 <= 1e-2 and max-abs <= 2e-2."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import moe
from gpu_common import FFN_MAX_ABS, FFN_REL_L2, layer_inputs, max_abs, rel_l2, to_f64, to_torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ew():
    import paper_2508_17624_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def _dense_pool(cfg, inp, poison=True):
    """The virtual weight tensors as plain device tensors [P, ...]; slots that hold no expert are
    filled with NaN so that any read of them shows up in the output."""
    dt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
    fill = float("nan") if poison else 0.0
    w13 = torch.full((cfg.P, 2 * cfg.I, cfg.H), fill, dtype=dt, device="cuda")
    w2 = torch.full((cfg.P, cfg.H, cfg.I), fill, dtype=dt, device="cuda")
    w13[:cfg.M] = to_torch(inp["base"][0]); w2[:cfg.M] = to_torch(inp["base"][1])
    for a, (a13, a2) in enumerate(inp["adapters"]):
        s0 = cfg.M + a * cfg.E_max
        if len(a13):
            w13[s0:s0 + len(a13)] = to_torch(a13); w2[s0:s0 + len(a2)] = to_torch(a2)
    return w13, w2


def _oracle_layer(cfg, inp, logits, aid=None):
    return moe.moe_layer(inp["x"], logits, inp["aid"] if aid is None else aid, cfg.k, cfg.M, cfg.N, cfg.E_max,
                         inp["tuned"], inp["base"], inp["adapters"], inp["shared"])


SMALL_BF16 = wl.get_config(1).with_(index=51, H=256, I=128, T=96, M=8, N=3, E_max=4, k=3, S=2, tuned_lo=0, tuned_hi=4,
                                    weight_std=0.04)   # keeps outputs O(0.5), like the full-size layer


@pytest.fixture
def ffn_path(ew, request):
    """Forces one of the bf16 kernels (1 = register streaming, 2 = tiled GEMM, 3 = LDS-direct streaming), then restores automatic."""
    ew.binding.tune_ffn(path=request.param)
    yield request.param
    ew.binding.tune_ffn()


@pytest.mark.parametrize("ffn_path", [1, 2, 3], indirect=True, ids=["stream", "gemm", "ws"])
@pytest.mark.parametrize("cfg", [SMALL_BF16, SMALL_BF16.with_(index=52, T=5, k=2), SMALL_BF16.with_(index=53, T=700, H=384, I=256)],
                         ids=["t96", "t5", "t700"])
def test_grouped_ffn_bf16_small(ew, cfg, ffn_path):
    """Several slots, empty slots, slots with more rows than one tile (t700), NaN padding; both kernels."""
    inp = layer_inputs(cfg)
    logits = moe.gate_logits(inp["x"], inp["Wg"])
    ref = _oracle_layer(cfg, inp, logits)
    w13, w2 = _dense_pool(cfg, inp)
    x = to_torch(inp["x"])
    dev = lambda a: torch.from_numpy(a).cuda()
    y = ew.moe_grouped_ffn(x, cfg.k, cfg.I, cfg.P, dev(ref["counts"]), dev(ref["offsets"]), dev(ref["pair_of_row"]), w13, w2)
    got = to_f64(y)
    assert np.isfinite(got).all(), "a slot without an expert was read"
    assert rel_l2(got, ref["y_sorted"]) <= FFN_REL_L2 and max_abs(got, ref["y_sorted"]) <= FFN_MAX_ABS
    # per-row check so one bad row cannot hide in the norm
    rows = np.linalg.norm(got - ref["y_sorted"], axis=1) / (np.linalg.norm(ref["y_sorted"], axis=1) + 1e-6)
    assert rows.max() <= 3e-2
    # un-permute with shared experts
    sh13, sh2 = to_torch(inp["shared"][0]), to_torch(inp["shared"][1])
    T, S = cfg.T, cfg.S
    shc = torch.full((S,), T, dtype=torch.int32, device="cuda")
    sho = (torch.arange(S + 1, dtype=torch.int32) * T).cuda()
    shp = (torch.arange(S * T, dtype=torch.int32) % T).cuda()
    ysh = ew.moe_grouped_ffn(x, 1, cfg.I, S, shc, sho, shp, sh13, sh2, num_rows=S * T)
    ref_sh = np.stack([moe.expert_ffn(inp["x"], inp["shared"][0][s], inp["shared"][1][s]) for s in range(S)])
    assert rel_l2(to_f64(ysh).reshape(S, T, -1), ref_sh) <= FFN_REL_L2
    out = ew.moe_unpermute(y, dev(ref["row_of_pair"]), dev(ref["w"].astype(np.float32)), ysh)
    assert rel_l2(to_f64(out), ref["out"]) <= FFN_REL_L2 and max_abs(to_f64(out), ref["out"]) <= FFN_MAX_ABS


@pytest.mark.parametrize("nf", [0, 8, 4, 1], ids=["auto", "nf8", "nf4", "nf1"])
def test_grouped_ffn_work_plan_edges(ew, nf):
    """The device-built work plan at its limits: 2048 slots, hundreds of them active (more than 64 entries per
    list), counts on every chunking boundary (1, 31..33, 255..257, 511..513, 700 rows), slots of more than eight
    chunks, which the plan cuts into several entries (2049, 2100, 4100 rows), first and last slot in use, every
    kernel shape.  Rows come straight from x (k = 1, shuffled row map)."""
    rng = np.random.default_rng(77)
    P, H, I = 2048, 128, 128
    counts = np.zeros(P, np.int32)
    special = [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 700, 2049, 2100, 4100]
    slots = rng.choice(np.arange(1, P - 1), size=len(special) + 560, replace=False)
    counts[slots[:len(special)]] = special
    counts[slots[len(special):]] = rng.integers(1, 24, size=560)
    counts[0], counts[P - 1] = 5, 40
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    rows = int(offsets[-1])
    por = rng.permutation(rows).astype(np.int32)
    x = torch.from_numpy(rng.standard_normal((rows, H), dtype=np.float32)).cuda().bfloat16()
    w13 = (torch.from_numpy(rng.standard_normal((P, 2 * I, H), dtype=np.float32)) * 0.08).cuda().bfloat16()
    w2 = (torch.from_numpy(rng.standard_normal((P, H, I), dtype=np.float32)) * 0.08).cuda().bfloat16()
    dev = lambda a: torch.from_numpy(a).cuda()
    ew.binding.tune_ffn(path=3 if nf else 0, ws_frags=nf)
    try:
        y = ew.moe_grouped_ffn(x, 1, I, P, dev(counts), dev(offsets), dev(por), w13, w2, num_rows=rows)
        torch.cuda.synchronize()
    finally:
        ew.binding.tune_ffn()
    got, xs = to_f64(y), to_f64(x)
    check = list(slots[:len(special)]) + [0, P - 1] + list(rng.choice(slots[len(special):], 40, replace=False))
    for s in check:
        r0, r1 = offsets[s], offsets[s + 1]
        ref = moe.expert_ffn(xs[por[r0:r1]], to_f64(w13[s]), to_f64(w2[s]))
        assert rel_l2(got[r0:r1], ref) <= FFN_REL_L2 and max_abs(got[r0:r1], ref) <= FFN_MAX_ABS, f"slot {s} ({counts[s]} rows)"
    assert np.isfinite(got).all()


@pytest.mark.gpu
@pytest.mark.parametrize("T,k,P,S,nf", [(37, 2, 24, 3, 2), (300, 4, 40, 2, 4), (300, 4, 40, 2, 8), (64, 6, 96, 1, 2), (1100, 2, 6, 2, 8),
                                        (300, 4, 40, 2, 0), (6000, 2, 14, 2, 8)],
                         ids=["ragged37", "t300-nf4", "t300-nf8", "decode64", "few-slots", "t300-auto", "large-slots"])
def test_grouped_ffn_with_shared(ew, T, k, P, S, nf):
    """Routed + shared experts in one launch: every row against the oracle's expert FFN, and -- when all calls are made
    with one kernel shape (nf > 0; the shapes walk the contraction in different orders) -- bit for bit against two plain
    moe_grouped_ffn calls (the same kernels on the same rows)."""
    rng = np.random.default_rng(100 + T)
    H, I = 256, 128
    ids = np.stack([rng.choice(P, k, replace=False) for _ in range(T)]).astype(np.int32)
    ids[:, 0] = np.where(rng.random(T) < 0.5, 3, ids[:, 0])               # one crowded slot; a repeat inside a token is fine here
    flat = ids.reshape(-1)
    por = np.argsort(flat, kind="stable").astype(np.int32)
    counts = np.bincount(flat, minlength=P).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    bf = lambda *shape, scale=1.0: (torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)) * scale).cuda().bfloat16()
    x, w13, w2, s13, s2 = bf(T, H), bf(P, 2 * I, H, scale=0.05), bf(P, H, I, scale=0.05), bf(S, 2 * I, H, scale=0.05), bf(S, H, I, scale=0.05)
    ew.binding.tune_ffn(path=3 if nf else 0, ws_frags=nf)
    try:
        y = ew.binding.moe_grouped_ffn_with_shared(x, k, I, P, dev(counts), dev(offsets), dev(por), w13, w2, s13, s2)
        y_routed = ew.moe_grouped_ffn(x, k, I, P, dev(counts), dev(offsets), dev(por), w13, w2)
        sh_counts = np.full(S, T, np.int32)
        sh_offsets = (np.arange(S + 1) * T).astype(np.int32)
        sh_por = (np.arange(S * T) % T).astype(np.int32)
        y_shared = ew.moe_grouped_ffn(x, 1, I, S, dev(sh_counts), dev(sh_offsets), dev(sh_por), s13, s2, num_rows=S * T)
        torch.cuda.synchronize()
    finally:
        ew.binding.tune_ffn()
    assert y.shape == (T * (k + S), H)
    if nf:
        assert torch.equal(y[:T * k], y_routed) and torch.equal(y[T * k:], y_shared)
    got, xs = to_f64(y), to_f64(x)
    for s in range(P):
        r0, r1 = offsets[s], offsets[s + 1]
        if r1 > r0:
            ref = moe.expert_ffn(xs[por[r0:r1] // k], to_f64(w13[s]), to_f64(w2[s]))
            assert rel_l2(got[r0:r1], ref) <= FFN_REL_L2 and max_abs(got[r0:r1], ref) <= FFN_MAX_ABS, f"slot {s}"
    for s in range(S):
        ref = moe.expert_ffn(xs, to_f64(s13[s]), to_f64(s2[s]))
        blk = got[T * k + s * T:T * k + (s + 1) * T]
        assert rel_l2(blk, ref) <= FFN_REL_L2 and max_abs(blk, ref) <= FFN_MAX_ABS, f"shared expert {s}"
    # limits: fp32 and S = 0 are refused
    with pytest.raises(ew.EWError):
        ew.binding.moe_grouped_ffn_with_shared(x.float(), k, I, P, dev(counts), dev(offsets), dev(por), w13.float(), w2.float(),
                                               s13.float(), s2.float())
    with pytest.raises(ew.EWError):
        ew.binding.moe_grouped_ffn_with_shared(x, k, I, P, dev(counts), dev(offsets), dev(por), w13, w2, s13[:0], s2[:0])


@pytest.mark.parametrize("T,k,E,N,S", [(64, 6, 64, 4, 2), (300, 4, 32, 2, 1), (40, 2, 192, 15, 0), (3000, 2, 16, 3, 2), (3000, 1, 16, 3, 1), (300, 9, 16, 3, 2),
                                       (400, 6, 64, 57, 1), (400, 6, 64, 117, 0), (3000, 2, 18, 3, 2), (131100, 2, 16, 3, 1)],
                         ids=["decode64", "one-block-300", "plan-launch-P1632", "multi-block-3000", "one-choice", "nine-choices", "P520", "P1000",
                              "P42-column-scan", "2^18-pairs-column-scan"])
def test_permutation_call_can_write_the_ffn_plan(ew, T, k, E, N, S):
    """moe_route_reroute_permute_plan + moe_grouped_ffn_planned against the plain pair of calls: same permutation, same
    FFN output bit for bit (the plan is the same plan, whoever writes it): by the single block, by a launch of its own, and by a block
    of each scatter kernel, with the histogram's columns summed there and with a column scan before it."""
    B = ew.binding
    rng = np.random.default_rng(T + E)
    H, I, E_max = 256, 128, 8 if E < 100 else 96
    P = E + N * E_max
    dev = lambda a: torch.from_numpy(a).cuda()
    logits = dev(rng.standard_normal((T, E), dtype=np.float32))
    aid_np = rng.integers(0, N + 1, T).astype(np.int32)
    tuned = [np.sort(rng.choice(E, E_max, replace=False)) for _ in range(N)]
    emap = dev(moe.build_expert_map(E, N, E_max, tuned).astype(np.int32))
    aid = dev(aid_np)
    bf = lambda *shape: (torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)) * 0.05).cuda().bfloat16()
    x, w13, w2 = bf(T, H) * 20, bf(P, 2 * I, H), bf(P, H, I)
    s13, s2 = (bf(S, 2 * I, H), bf(S, H, I)) if S else (None, None)
    lib, st, i32 = B.lib(), B._stream(), dict(dtype=torch.int32, device="cuda")
    dt = B.EW_BF16

    def run(planned):
        ids, w = torch.empty((T, k), **i32), torch.empty((T, k), dtype=torch.float32, device="cuda")
        slot, counts, offsets = torch.empty((T, k), **i32), torch.empty(P, **i32), torch.empty(P + 1, **i32)
        por, rop = torch.empty(T * k, **i32), torch.empty(T * k, **i32)
        ws = B._workspace(lib.moe_reroute_permute_workspace_bytes(T, k, P), "cuda")
        ws_ffn = B._workspace(lib.moe_grouped_ffn_workspace_bytes(T, k + S, H, I, P + S, dt), "cuda")
        ws_ffn.fill_(0x5A)                                                  # whatever a previous call left there
        y = torch.empty((T * (k + S), H), dtype=torch.bfloat16, device="cuda")
        args = (logits.data_ptr(), aid.data_ptr(), emap.data_ptr(), T, E, k, N, P, 0, ids.data_ptr(), w.data_ptr(), slot.data_ptr(),
                counts.data_ptr(), offsets.data_ptr(), por.data_ptr(), rop.data_ptr(), B._ptr(ws), ws.numel() if ws is not None else 0)
        ffn = (x.data_ptr(), dt, T, k, H, I, P, S, counts.data_ptr(), offsets.data_ptr(), por.data_ptr(), w13.data_ptr(),
               w2.data_ptr(), B._ptr(s13), B._ptr(s2), y.data_ptr(), ws_ffn.data_ptr(), ws_ffn.numel(), st)
        if planned:
            B._check(lib.moe_route_reroute_permute_plan(*args, H, I, S, dt, ws_ffn.data_ptr(), ws_ffn.numel(), st))
            B._check(lib.moe_grouped_ffn_planned(*ffn))
        else:
            B._check(lib.moe_route_reroute_permute(*args, st))
            if S:
                B._check(lib.moe_grouped_ffn_with_shared(*ffn))
            else:
                B._check(lib.moe_grouped_ffn(*(ffn[:7] + ffn[8:13] + ffn[15:])))
        torch.cuda.synchronize()
        return ids, w, slot, counts, offsets, por, rop, y

    plain, planned = run(False), run(True)
    for name, a, b in zip(("ids", "w", "slot", "counts", "offsets", "pair_of_row", "row_of_pair", "y"), plain, planned):
        assert torch.equal(a, b), name
    # and the plain pair is the oracle's permutation
    ids_ref, _ = moe.route_topk(logits.cpu().numpy(), k)
    slot_ref = moe.reroute(ids_ref, aid_np, emap.cpu().numpy())
    counts_ref, offsets_ref, por_ref, rop_ref = moe.permute(slot_ref, P)
    np.testing.assert_array_equal(planned[5].cpu().numpy(), por_ref)
    np.testing.assert_array_equal(planned[3].cpu().numpy(), counts_ref)
    # fp32 has no plan
    with pytest.raises(ew.EWError):
        ws_ffn = B._workspace(lib.moe_grouped_ffn_workspace_bytes(T, k + S, H, I, P + S, B.EW_F32), "cuda")
        i = lambda *sh: torch.empty(sh, **i32)
        B._check(lib.moe_route_reroute_permute_plan(logits.data_ptr(), aid.data_ptr(), emap.data_ptr(), T, E, k, N, P, 0,
                                                    i(T, k).data_ptr(), torch.empty((T, k), device="cuda").data_ptr(),
                                                    i(T, k).data_ptr(), i(P).data_ptr(), i(P + 1).data_ptr(), i(T * k).data_ptr(),
                                                    i(T * k).data_ptr(), None, 0, H, I, S, B.EW_F32, ws_ffn.data_ptr(),
                                                    ws_ffn.numel(), st))


@pytest.mark.parametrize("T,k,P,S,nf", [(64, 6, 128, 2, 0), (256, 6, 384, 2, 0), (200, 4, 48, 0, 4), (31, 2, 300, 1, 1)],
                         ids=["decode64", "decode256", "nf4-no-shared", "nf1"])
def test_one_launch_for_both_products_equals_two(ew, T, k, P, S, nf):
    """Decode shapes run both products in one launch, second-product items waiting for the activation rows they read:
    bit for bit the two-launch result, on repeated calls (the completion counters are rebuilt by every plan)."""
    rng = np.random.default_rng(T * 3 + P)
    H, I = 512, 384
    ids = np.stack([rng.choice(P, k, replace=False) for _ in range(T)]).astype(np.int32)
    flat = ids.reshape(-1)
    por = np.argsort(flat, kind="stable").astype(np.int32)
    counts = np.bincount(flat, minlength=P).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    bf = lambda *shape, scale=1.0: (torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)) * scale).cuda().bfloat16()
    x, w13, w2 = bf(T, H), bf(P, 2 * I, H, scale=0.04), bf(P, H, I, scale=0.04)
    s13, s2 = (bf(S, 2 * I, H, scale=0.04), bf(S, H, I, scale=0.04)) if S else (None, None)

    def run(two_launches):
        ew.binding.tune_ffn(path=3 if nf else 0, ws_frags=nf, ws_two_launches=two_launches)
        try:
            if S:
                y = ew.binding.moe_grouped_ffn_with_shared(x, k, I, P, dev(counts), dev(offsets), dev(por), w13, w2, s13, s2)
            else:
                y = ew.moe_grouped_ffn(x, k, I, P, dev(counts), dev(offsets), dev(por), w13, w2)
            torch.cuda.synchronize()
        finally:
            ew.binding.tune_ffn()
        return y

    ref = run(True)
    for _ in range(3):
        assert torch.equal(run(False), ref)
    got, xs = to_f64(ref), to_f64(x)
    for s in np.nonzero(counts)[0][:12]:
        r0, r1 = offsets[s], offsets[s + 1]
        want = moe.expert_ffn(xs[por[r0:r1] // k], to_f64(w13[s]), to_f64(w2[s]))
        assert rel_l2(got[r0:r1], want) <= FFN_REL_L2 and max_abs(got[r0:r1], want) <= FFN_MAX_ABS, f"slot {s}"


@pytest.mark.parametrize("T,k,P,S,H,I", [(1500, 2, 6, 2, 640, 128), (1100, 2, 8, 2, 2176, 1408), (700, 3, 40, 0, 896, 256), (900, 4, 5, 1, 384, 1408)],
                         ids=["two-slabs", "more-units-than-cus", "thin-slots", "odd-hidden"])
def test_one_launch_of_the_many_rows_kernel_equals_two(ew, T, k, P, S, H, I):
    """k_ffn_big asked for by name: crowded slots cut into several chunks beside thin ones, hidden sizes that are an odd multiple
    of 128, two-slab contractions, fewer and more units than CUs.  One launch, whose second product reads rows that other
    workgroups have just stored, gives the bits of two launches on every one of several calls; some rows against the oracle."""
    rng = np.random.default_rng(T * 5 + H)
    ids = np.stack([rng.choice(P, k, replace=False) for _ in range(T)]).astype(np.int32)
    ids[:, 0] = np.where(rng.random(T) < 0.6, 1, ids[:, 0])               # a repeat inside a token is fine here
    flat = ids.reshape(-1)
    por = np.argsort(flat, kind="stable").astype(np.int32)
    counts = np.bincount(flat, minlength=P).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    bf = lambda *shape, scale=1.0: (torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)) * scale).cuda().bfloat16()
    x, w13, w2 = bf(T, H), bf(P, 2 * I, H, scale=0.02), bf(P, H, I, scale=0.02)
    s13, s2 = (bf(S, 2 * I, H, scale=0.02), bf(S, H, I, scale=0.02)) if S else (None, None)
    args = (dev(counts), dev(offsets), dev(por), w13, w2)

    def run(two_launches):
        ew.binding.tune_ffn(path=3, ws_frags=8, ws_two_launches=two_launches)
        try:
            return ew.moe_grouped_ffn_with_shared(x, k, I, P, *args, s13, s2) if S else ew.moe_grouped_ffn(x, k, I, P, *args)
        finally:
            ew.binding.tune_ffn()

    ref = run(True)
    for _ in range(4):
        assert torch.equal(run(False), ref)
    got, xs = to_f64(ref), to_f64(x)
    for s in (1, int(np.argmin(np.where(counts > 0, counts, T * k + 1)))):
        r0, r1 = offsets[s], offsets[s + 1]
        want = moe.expert_ffn(xs[por[r0:r1] // k], to_f64(w13[s]), to_f64(w2[s]))
        assert rel_l2(got[r0:r1], want) <= FFN_REL_L2 and max_abs(got[r0:r1], want) <= FFN_MAX_ABS, f"slot {s}"


@pytest.mark.parametrize("T,k,P,H,I", [(1200, 2, 270, 2048, 128), (1200, 2, 135, 2048, 256), (1200, 2, 90, 2048, 384), (1200, 2, 67, 2048, 512),
                                       (1500, 2, 6, 2048, 256), (1500, 2, 6, 256, 1408)],
                         ids=["2-slabs", "4-slabs", "6-slabs", "8-slabs", "4-slabs-crowded", "4-slabs-first-crowded"])
def test_many_rows_kernel_waits_for_rows_of_short_contractions(ew, T, k, P, H, I):
    """k_ffn_big where one product's units are much shorter than the other's, one test for each way its scheduling steps share the slabs
    of a short unit: slightly more units of the long first product than workgroups, so that those with one unit less run through many
    units of the second one while others still store (and crowded slots with fewer units than workgroups).  The activations are NaN
    before each call: a row read before it is stored shows.  One launch gives the bits of two, and some slots agree with the oracle."""
    rng = np.random.default_rng(H * 3 + I + P)
    flat = np.concatenate([np.arange(P), rng.integers(0, P, T * k - P)]).astype(np.int32)[rng.permutation(T * k)]  # (a repeat inside a token is fine)
    por = np.argsort(flat, kind="stable").astype(np.int32)
    counts = np.bincount(flat, minlength=P).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    g = torch.Generator(device="cuda").manual_seed(H + I)
    bf = lambda *shape, scale=1.0: torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16) * scale
    x, w13, w2 = bf(T, H), bf(P, 2 * I, H, scale=0.02), bf(P, H, I, scale=0.02)
    args = (x, k, I, P, dev(counts), dev(offsets), dev(por), w13, w2)
    ws = ew.binding._workspace(ew.lib().moe_grouped_ffn_workspace_bytes(T, k, H, I, P, ew.EW_BF16), "cuda")

    def run(two_launches):
        ws.fill_(0xFF)
        ew.binding.tune_ffn(path=3, ws_frags=8, ws_two_launches=two_launches)
        try:
            return ew.moe_grouped_ffn(*args, ws=ws)
        finally:
            ew.binding.tune_ffn()

    ref = run(True)
    for _ in range(4):
        assert torch.equal(run(False), ref)
    got, xs = to_f64(ref), to_f64(x)
    for s in (0, int(np.argmax(counts)), P - 1):
        r0, r1 = offsets[s], offsets[s + 1]
        want = moe.expert_ffn(xs[por[r0:r1] // k], to_f64(w13[s]), to_f64(w2[s]))
        assert rel_l2(got[r0:r1], want) <= FFN_REL_L2 and max_abs(got[r0:r1], want) <= FFN_MAX_ABS, f"slot {s}"


@pytest.mark.parametrize("T", [16, 256], ids=["few-rows", "many-rows"])
def test_a_wait_given_up_writes_nan(ew, T):
    """One slot with fewer first-product units than workgroups: those left over start with units of the second product, whose
    activation rows cannot be there at their first look.  Allowed one look only, they give up: what they write is NaN, everything
    else has the bits of the undisturbed call, and so has the whole next call."""
    k, P, H, I = 1, 1, 2048, 1408
    rng = np.random.default_rng(T)
    i32 = lambda *v: torch.tensor(v, dtype=torch.int32, device="cuda")
    bf = lambda *shape, scale=1.0: (torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)) * scale).cuda().bfloat16()
    x, w13, w2 = bf(T, H), bf(P, 2 * I, H, scale=0.02), bf(P, H, I, scale=0.02)

    def run(looks):
        ew.binding.tune_ffn(ws_wait_ticks=looks)
        try:
            return ew.moe_grouped_ffn(x, k, I, P, i32(T), i32(0, T), None, w13, w2)
        finally:
            ew.binding.tune_ffn()

    ref = run(-1)
    assert torch.isfinite(ref.float()).all()
    got = run(1)
    given_up = torch.isnan(got)
    assert given_up.any() and torch.equal(got[~given_up], ref[~given_up])
    assert torch.equal(run(-1), ref)


def test_one_launch_equals_two_on_random_decode_shapes(ew):
    """Twenty random decode-sized calls (token count, top-k, slots, shared experts, skew all drawn): the one-launch
    result equals the two-launch result bit for bit every time, with and without a row map."""
    rng = np.random.default_rng(20250817)
    H, I = 256, 128
    dev = lambda a: torch.from_numpy(a).cuda()
    bf = lambda *shape, scale=1.0: (torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)) * scale).cuda().bfloat16()
    for case in range(20):
        T = int(rng.integers(1, 300))
        k = int(rng.integers(1, 7))
        P = int(rng.integers(k, 200))
        S = int(rng.integers(0, 3))
        hot = rng.random() < 0.5
        ids = np.stack([rng.choice(P, k, replace=False) for _ in range(T)]).astype(np.int32)
        if hot:
            ids[:, 0] = np.where(rng.random(T) < 0.7, 0, ids[:, 0])          # most tokens also visit slot 0 (a repeat is fine here)
        flat = ids.reshape(-1)
        por = np.argsort(flat, kind="stable").astype(np.int32)
        counts = np.bincount(flat, minlength=P).astype(np.int32)
        offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
        x, w13, w2 = bf(T, H), bf(P, 2 * I, H, scale=0.05), bf(P, H, I, scale=0.05)
        s13, s2 = (bf(S, 2 * I, H, scale=0.05), bf(S, H, I, scale=0.05)) if S else (None, None)
        outs = []
        for two in (True, False, False):
            ew.binding.tune_ffn(ws_two_launches=two)
            try:
                if S:
                    y = ew.binding.moe_grouped_ffn_with_shared(x, k, I, P, dev(counts), dev(offsets), dev(por), w13, w2, s13, s2)
                else:
                    y = ew.moe_grouped_ffn(x, k, I, P, dev(counts), dev(offsets), dev(por), w13, w2)
                torch.cuda.synchronize()
            finally:
                ew.binding.tune_ffn()
            outs.append(y)
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2]), f"case {case}: T={T} k={k} P={P} S={S} hot={hot}"
        assert torch.isfinite(outs[0].float()).all()
        s = int(np.argmax(counts))
        r0, r1 = offsets[s], offsets[s + 1]
        want = moe.expert_ffn(to_f64(x)[por[r0:r1] // k], to_f64(w13[s]), to_f64(w2[s]))
        got = to_f64(outs[1])[r0:r1]
        assert rel_l2(got, want) <= FFN_REL_L2 and max_abs(got, want) <= FFN_MAX_ABS, f"case {case}: slot {s}"


def test_unpermute_exact_combination(ew):
    """moe_unpermute alone, f32: inputs chosen so fp32 arithmetic is exact."""
    rng = np.random.default_rng(0)
    T, k, H, S = 37, 3, 64, 2
    y = rng.integers(-8, 9, size=(T * k, H)).astype(np.float32)
    w = rng.choice([0.25, 0.5, 1.0, 2.0], size=(T, k)).astype(np.float32)
    sh = rng.integers(-4, 5, size=(S, T, H)).astype(np.float32)
    rop = rng.permutation(T * k).astype(np.int32)
    ref = moe.unpermute(y, rop, w, sh.sum(0))
    dev = lambda a: torch.from_numpy(a).cuda()
    np.testing.assert_array_equal(to_f64(ew.moe_unpermute(dev(y), dev(rop), dev(w), dev(sh))), ref)
    np.testing.assert_array_equal(to_f64(ew.moe_unpermute(dev(y), dev(rop), dev(w), None)), moe.unpermute(y, rop, w))
    yb, shb = dev(y).bfloat16(), dev(sh).bfloat16()                        # small integers: exact in bf16 too
    got = to_f64(ew.moe_unpermute(yb, dev(rop), dev(w), shb))
    np.testing.assert_allclose(got, ref, rtol=2 ** -8)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,k,H,S", [(37, 3, 2048, 2), (5, 6, 4104, 0), (64, 2, 256, 1)])
def test_unpermute_rmsnorm_equals_the_two_calls(ew, dtype, T, k, H, S):
    """The fused combine + normalisation: bit for bit the two separate calls, and the oracle's values."""
    rng = np.random.default_rng(T * 7 + H)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev = lambda a: torch.from_numpy(a).cuda()
    y = dev(rng.standard_normal((T * k, H), dtype=np.float32)).to(td)
    w = dev(rng.random((T, k), dtype=np.float32))
    sh = dev(rng.standard_normal((S, T, H), dtype=np.float32)).to(td) if S else None
    res = dev(rng.standard_normal((T, H), dtype=np.float32)).to(td)
    rop_np = rng.permutation(T * k).astype(np.int32)
    rop, eps = dev(rop_np), 1e-6
    out2 = ew.moe_unpermute(y, rop, w, sh, residual=res)
    normed2 = ew.binding.moe_rmsnorm(out2, eps)
    out1, normed1 = ew.binding.moe_unpermute_rmsnorm(y, rop, w, eps, shared_out=sh, residual=res)
    torch.cuda.synchronize()
    assert torch.equal(out1, out2) and torch.equal(normed1, normed2)
    ref = moe.unpermute(to_f64(y), rop_np, w.cpu().numpy(), to_f64(sh).sum(0) if S else None) + to_f64(res)
    tol = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -20
    assert max_abs(to_f64(out1), ref) <= tol * np.abs(ref).max()
    ref_n = moe.rmsnorm(to_f64(out1), eps)
    assert max_abs(to_f64(normed1), ref_n) <= tol * np.abs(ref_n).max()
    with pytest.raises(ew.EWError):
        ew.binding.moe_unpermute_rmsnorm(y, rop, w, eps, shared_out=sh, out=out1, normed_out=out1)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,k,H,S,res", [(11, 1, 8, 0, False), (1, 2, 2048, 1, True), (11, 3, 2056, 2, False), (256, 4, 1016, 3, True),
                                         (257, 4, 1016, 3, True), (11, 5, 64, 0, True), (11, 6, 2048, 2, True), (11, 7, 4096, 5, False),
                                         (11, 8, 1544, 1, False), (11, 9, 2048, 2, True), (11, 64, 72, 3, False)])
def test_unpermute_every_width(ew, dtype, T, k, H, S, res):
    """Every number of experts per token that has a kernel of its own and two that do not, both sides of the token count up to
    which those kernels run, fewer and more shared rows than are loaded ahead, rows shorter and longer than a workgroup's step.
    Small integers and powers of two: exact in fp32, one rounding in bf16."""
    rng = np.random.default_rng(k * 100 + S)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev = lambda a: torch.from_numpy(a).cuda()
    y = rng.integers(-8, 9, size=(T * k, H)).astype(np.float32)
    w = rng.choice([0.25, 0.5, 1.0, 2.0], size=(T, k)).astype(np.float32)
    sh = rng.integers(-4, 5, size=(S, T, H)).astype(np.float32)
    r = rng.integers(-4, 5, size=(T, H)).astype(np.float32)
    rop = rng.permutation(T * k).astype(np.int32)
    ref = moe.unpermute(y, rop, w, sh.sum(0) if S else None) + (r if res else 0)
    got = ew.moe_unpermute(dev(y).to(td), dev(rop), dev(w), dev(sh).to(td) if S else None, residual=dev(r).to(td) if res else None)
    want = torch.from_numpy(np.ascontiguousarray(ref)).to(torch.float32).to(td)
    assert torch.equal(got.cpu(), want)


@pytest.mark.parametrize("cfg_index", [0, 1])
def test_gate_logits(ew, cfg_index):
    cfg = wl.get_config(cfg_index).with_(gate_bias=2.0)
    tuned = wl.tuned_sets(cfg)
    x, Wg, aid = wl.tokens(cfg), wl.gate_weight(cfg), wl.adapter_ids(cfg)
    bias = wl.logit_bias_table(cfg, tuned)
    dev = lambda a: torch.from_numpy(a).cuda()
    got = ew.moe_gate_logits(to_torch(x), dev(Wg), dev(aid), dev(bias)).cpu().numpy()
    ref = moe.gate_logits(x, Wg, aid, bias)
    np.testing.assert_allclose(got, ref, rtol=1e-4, atol=2e-5)
    got0 = ew.moe_gate_logits(to_torch(x), dev(Wg)).cpu().numpy()
    np.testing.assert_allclose(got0, moe.gate_logits(x, Wg), rtol=1e-4, atol=2e-5)


GATE_CASES = [(1, 1, 128), (17, 3, 640), (128, 64, 512), (129, 64, 512), (300, 37, 1024), (512, 64, 512), (1030, 96, 384), (2048, 64, 512),
              (2100, 50, 640), (4096, 64, 512), (4100, 70, 512), (9000, 33, 128), (129, 64, 640), (500, 64, 640), (1000, 64, 512), (1000, 64, 640),
              (4096, 64, 640)]


def _gate_tile(T, E, H):
    """(waves, token tiles, experts) of the workgroup that moe_gate_logits picks: the smallest whose grid is one per CU of 256."""
    cdiv = lambda a, b: -(-a // b)
    tiles = [(1, 2), (1, 4), (1, 8), (1, 16), (2, 16), (4, 16), (4, 32)]
    return (16 if H % 512 == 0 else 4,) + next((t for t in tiles if cdiv(T, 16 * t[0]) * cdiv(E, t[1]) <= 256), tiles[-1])


def test_gate_logits_cases_cover_every_tile():
    tiles = {(nw,) + t for nw in (4, 16) for t in [(1, 2), (1, 4), (1, 8), (1, 16), (2, 16), (4, 16), (4, 32)]}
    assert {_gate_tile(*c) for c in GATE_CASES} == tiles


@pytest.mark.parametrize("T,E,H", GATE_CASES)
def test_gate_logits_tiles(ew, T, E, H):
    """Every tile of the matrix-core kernel with both wave counts, and sizes that fill a tile's tokens and experts only partly.  The
    bf16 head and tail of a gate weight leave 2^-17 of it; with sums of a few dozen such products that stays below the bound."""
    g = torch.Generator(device="cuda").manual_seed(T + E + H)
    x = torch.randn((T, H), generator=g, device="cuda").to(torch.bfloat16)
    Wg = torch.randn((E, H), generator=g, device="cuda") * 0.02
    aid = torch.randint(0, 3, (T,), generator=g, device="cuda", dtype=torch.int32)
    bias = torch.randn((3, E), generator=g, device="cuda")
    ref = x.double() @ Wg.double().T
    np.testing.assert_allclose(ew.moe_gate_logits(x, Wg).cpu().numpy(), ref.cpu().numpy(), rtol=1e-4, atol=2e-5)
    got = ew.moe_gate_logits(x, Wg, aid, bias).cpu().numpy()
    np.testing.assert_allclose(got, (ref + bias.double()[aid.long()]).cpu().numpy(), rtol=1e-4, atol=2e-5)


@pytest.mark.parametrize("dtype,T,E,H", [("f32", 1, 1, 4), ("f32", 5, 7, 252), ("f32", 64, 8, 256), ("f32", 6, 9, 260), ("f32", 3, 130, 1028),
                                         ("bf16", 5, 8, 64), ("bf16", 9, 21, 324)])
def test_gate_logits_without_matrix_cores(ew, dtype, T, E, H):
    """Experts that do not fill a group of eight, widths that do not fill a wave's loads, with and without the bias.  Plain fp32 sums
    of at most 1028 products of deviation 0.02: a few dozen roundings of 2^-24 of sums below 4."""
    g = torch.Generator(device="cuda").manual_seed(T + E + H)
    x = torch.randn((T, H), generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    Wg = torch.randn((E, H), generator=g, device="cuda") * 0.02
    aid = torch.randint(0, 3, (T,), generator=g, device="cuda", dtype=torch.int32)
    bias = torch.randn((3, E), generator=g, device="cuda")
    ref = x.double() @ Wg.double().T
    np.testing.assert_allclose(ew.moe_gate_logits(x, Wg).cpu().numpy(), ref.cpu().numpy(), rtol=1e-5, atol=5e-6)
    got = ew.moe_gate_logits(x, Wg, aid, bias).cpu().numpy()
    np.testing.assert_allclose(got, (ref + bias.double()[aid.long()]).cpu().numpy(), rtol=1e-5, atol=5e-6)


def _run_layer_through_pool(ew, cfg, inp, logits, flags=0, aid=None):
    from paper_2508_17624_amd.layer import MoELayer, load_layer
    dt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
    el = 2 if cfg.dtype == "bf16" else 4
    pool = ew.ExpertPool(1, cfg.M, cfg.N, cfg.E_max, 2 * cfg.I * cfg.H * el, cfg.H * cfg.I * el, flags=flags)
    t = lambda a: torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a)   # host tensors: H2D copy inside map
    load_layer(pool, 0, (t(inp["base"][0]), t(inp["base"][1])), [(t(a), t(b)) for a, b in inp["adapters"]], inp["tuned"])
    emap = pool.expert_map_host(0).numpy()
    np.testing.assert_array_equal(emap, moe.build_expert_map(cfg.M, cfg.N, cfg.E_max, inp["tuned"]))
    sh13, sh2 = (to_torch(inp["shared"][0]), to_torch(inp["shared"][1])) if cfg.S else (None, None)
    layer = MoELayer(pool, 0, torch.from_numpy(inp["Wg"]).cuda(), sh13, sh2, cfg.k, cfg.I, cfg.T, dt)
    aid_t = torch.from_numpy(inp["aid"] if aid is None else aid).cuda()
    out = layer.forward(to_torch(inp["x"]), aid_t, torch.from_numpy(logits).cuda()).clone()
    torch.cuda.synchronize()
    return pool, layer, out


def test_layer_c0_f32(ew):
    """Config 0 end to end in fp32 through a VMM pool."""
    cfg = wl.get_config(0)
    inp = layer_inputs(cfg)
    logits = moe.gate_logits(inp["x"], inp["Wg"])
    ref = _oracle_layer(cfg, inp, logits)
    pool, layer, out = _run_layer_through_pool(ew, cfg, inp, logits)
    np.testing.assert_array_equal(layer.ids.cpu().numpy(), ref["ids"])
    np.testing.assert_array_equal(layer.slot.cpu().numpy(), ref["slot"])
    np.testing.assert_array_equal(layer.por.cpu().numpy(), ref["pair_of_row"])
    assert rel_l2(to_f64(out), ref["out"]) <= 1e-5                          # fp32 arithmetic, K <= 256
    assert rel_l2(to_f64(layer.y), ref["y_sorted"]) <= 1e-5
    st = pool.stats()
    assert st["experts_loaded"] == cfg.M + sum(len(J) for J in inp["tuned"])
    pool.close()


def test_layer_c1_bf16_vmm_and_merge_equivalence(ew):
    """Config 1 (DeepSeek-V2-Lite decode shape) end to end through a VMM pool; also against the
    merged-model path of the oracle (the paper's accuracy claim) and a base-only batch."""
    cfg = wl.get_config(1)
    inp = layer_inputs(cfg)
    logits = moe.gate_logits(inp["x"], inp["Wg"])
    ref = _oracle_layer(cfg, inp, logits)
    pool, layer, out = _run_layer_through_pool(ew, cfg, inp, logits)
    for name, got in (("ids", layer.ids), ("slot", layer.slot), ("counts", layer.counts), ("offsets", layer.offsets),
                      ("pair_of_row", layer.por), ("row_of_pair", layer.rop)):
        np.testing.assert_array_equal(got.cpu().numpy().reshape(ref[name].shape), ref[name], err_msg=name)
    got = to_f64(out)
    assert rel_l2(to_f64(layer.y), ref["y_sorted"]) <= FFN_REL_L2 and max_abs(to_f64(layer.y), ref["y_sorted"]) <= FFN_MAX_ABS
    assert rel_l2(got, ref["out"]) <= FFN_REL_L2 and max_abs(got, ref["out"]) <= FFN_MAX_ABS
    merged = moe.merged_model_layer(inp["x"], logits, inp["aid"], cfg.k, cfg.M, inp["tuned"], inp["base"], inp["adapters"], inp["shared"])
    assert rel_l2(got, merged) <= FFN_REL_L2
    # base-only batch on the same pool: slots == ids, adapter slots untouched
    aid0 = np.zeros_like(inp["aid"])
    out0 = layer.forward(to_torch(inp["x"]), torch.from_numpy(aid0).cuda(), torch.from_numpy(logits).cuda()).clone()
    ref0 = _oracle_layer(cfg, inp, logits, aid0)
    assert torch.equal(layer.slot, layer.ids) and int(layer.counts[cfg.M:].sum()) == 0
    assert rel_l2(to_f64(out0), ref0["out"]) <= FFN_REL_L2
    # gate kernel feeding the fused router: ids agree wherever the k-th/(k+1)-th margin is clear
    lg = ew.moe_gate_logits(to_torch(inp["x"]), torch.from_numpy(inp["Wg"]).cuda())
    srt = np.sort(logits, axis=1)[:, ::-1]
    clear = (srt[:, :cfg.k] - srt[:, 1:cfg.k + 1]).min(axis=1) > 1e-4
    ids_g, _ = ew.moe_route_topk(lg, cfg.k)
    np.testing.assert_array_equal(ids_g.cpu().numpy()[clear], ref["ids"][clear])
    pool.close()


@pytest.fixture(scope="module")
def c2(ew):
    """Configuration 2 loaded once for the tests below: inputs, VMM pool, layer, oracle-side logits."""
    cfg = wl.get_config(2)
    inp = layer_inputs(cfg)
    logits = moe.gate_logits(inp["x"], inp["Wg"], inp["aid"], inp["bias"])
    pool, layer, out = _run_layer_through_pool(ew, cfg, inp, logits)
    yield dict(cfg=cfg, inp=inp, logits=logits, pool=pool, layer=layer, out=out)
    pool.close()


def _compare_full(cfg, layer, out, ref, T, what):
    """Integer stages bit for bit, combine weights, then every FFN row and every output row."""
    n = T * cfg.k
    for name, got in (("ids", layer.ids[:T]), ("slot", layer.slot[:T]), ("counts", layer.counts), ("offsets", layer.offsets),
                      ("pair_of_row", layer.por[:n]), ("row_of_pair", layer.rop[:n])):
        np.testing.assert_array_equal(got.cpu().numpy().reshape(ref[name].shape), ref[name], err_msg=f"{what}: {name}")
    np.testing.assert_allclose(layer.w[:T].cpu().numpy(), ref["w"], rtol=2e-5, atol=1e-9)
    y = to_f64(layer.y[:n])
    assert np.isfinite(y).all(), f"{what}: a slot without an expert was read"
    assert rel_l2(y, ref["y_sorted"]) <= FFN_REL_L2 and max_abs(y, ref["y_sorted"]) <= FFN_MAX_ABS, what
    # row by row, so that one wrong row of one chunk, fragment or feature group cannot hide in the norm
    err = np.linalg.norm(y - ref["y_sorted"], axis=1) / (np.linalg.norm(ref["y_sorted"], axis=1) + 1e-3)
    assert err.max() <= 3e-2, f"{what}: sorted row {int(err.argmax())} is off by {err.max():.3e}"
    got = to_f64(out)
    assert rel_l2(got, ref["out"]) <= FFN_REL_L2 and max_abs(got, ref["out"]) <= FFN_MAX_ABS, what
    err = np.linalg.norm(got - ref["out"], axis=1) / (np.linalg.norm(ref["out"], axis=1) + 1e-3)
    assert err.max() <= 3e-2, f"{what}: token {int(err.argmax())} is off by {err.max():.3e}"


def test_layer_c2_full_size(ew, c2):
    """Configuration 2 at full size (8192-token prefill, 20 adapters, Zipf classes, biased gates), in the launch
    configuration the benchmark times: every integer output bit for bit, every one of the 49 152 FFN rows and 8192
    output rows against the oracle."""
    cfg, inp, logits, layer = c2["cfg"], c2["inp"], c2["logits"], c2["layer"]
    ref = _oracle_layer(cfg, inp, logits)
    _compare_full(cfg, layer, c2["out"], ref, cfg.T, "c2")
    assert int((ref["counts"] > 0).sum()) > 200                      # the regime of many active slots
    # the gate kernel at this shape (bias per class included)
    lg = ew.moe_gate_logits(to_torch(inp["x"]), torch.from_numpy(inp["Wg"]).cuda(), torch.from_numpy(inp["aid"]).cuda(),
                            torch.from_numpy(inp["bias"]).cuda()).cpu().numpy()
    np.testing.assert_allclose(lg, logits, rtol=1e-4, atol=3e-5)
    # base-only traffic on the same pool (what the overhead is measured against)
    aid0 = np.zeros_like(inp["aid"])
    logits0 = moe.gate_logits(inp["x"], inp["Wg"])
    out0 = layer.forward(to_torch(inp["x"]), torch.from_numpy(aid0).cuda(), torch.from_numpy(logits0).cuda()).clone()
    torch.cuda.synchronize()
    _compare_full(cfg, layer, out0, _oracle_layer(cfg, inp, logits0, aid0), cfg.T, "c2 base-only")


@pytest.mark.parametrize("T,n_adapters,alpha", [(512, 5, 1.0), (512, 5, 0.1), (512, 20, 1.0), (512, 20, 0.1),
                                                (2048, 5, 1.0), (2048, 5, 0.1), (2048, 20, 1.0), (2048, 20, 0.1)])
def test_second_workload_parity(ew, c2, T, n_adapters, alpha):
    """Chunked-prefill sizes with skewed adapter popularity on the configuration-2 layer (Sec. 5.1: per-adapter
    request shares from a power law with shape alpha; Sec. 5.2: 5 to 20 adapters), the points the benchmark's
    sweep times: all outputs against the oracle."""
    cfg, inp, layer = c2["cfg"], c2["inp"], c2["layer"]
    aid = wl.adapter_ids_powerlaw(cfg, T, n_adapters, alpha)
    assert aid.min() >= 1 and aid.max() <= n_adapters
    sub = dict(inp, x=inp["x"][:T], aid=aid)
    logits = moe.gate_logits(sub["x"], inp["Wg"], aid, inp["bias"])
    out = layer.forward(to_torch(sub["x"]), torch.from_numpy(aid).cuda(), torch.from_numpy(logits).cuda()).clone()
    torch.cuda.synchronize()
    ref = _oracle_layer(cfg, sub, logits)
    _compare_full(cfg, layer, out, ref, T, f"T={T} n={n_adapters} alpha={alpha}")


def test_layer_c1_padded_pool_matches_oracle_and_vmm(ew):
    """The padding approach of Sec. 3.1 on the real VMM backend (every slot backed): same outputs as the oracle, and
    bit-identical to the sparse virtual tensor's (the kernels never learn which pool they run on)."""
    cfg = wl.get_config(1)
    inp = layer_inputs(cfg)
    logits = moe.gate_logits(inp["x"], inp["Wg"])
    ref = _oracle_layer(cfg, inp, logits)
    outs, stats = {}, {}
    for mode, flags in (("vmm", ew.EW_POOL_VMM), ("padded", ew.EW_POOL_PADDED)):
        pool, layer, out = _run_layer_through_pool(ew, cfg, inp, logits, flags=flags)
        _compare_full(cfg, layer, out, ref, cfg.T, mode)
        outs[mode], stats[mode] = (out, layer.y[:cfg.T * cfg.k].clone()), pool.stats()
        pool.close()
    assert torch.equal(outs["vmm"][0], outs["padded"][0]) and torch.equal(outs["vmm"][1], outs["padded"][1])
    el = 2 * 3 * cfg.H * cfg.I
    assert stats["padded"]["pages_mapped"] * stats["padded"]["page_bytes"] >= cfg.P * el
    assert stats["vmm"]["pages_mapped"] < stats["padded"]["pages_mapped"]
    assert stats["vmm"]["f_mem"] == pytest.approx(cfg.P / (cfg.M + sum(len(J) for J in inp["tuned"])))


def test_ffn_argument_errors(ew):
    x = torch.zeros((4, 100), dtype=torch.bfloat16, device="cuda")
    c = torch.zeros(2, dtype=torch.int32, device="cuda")
    with pytest.raises(ew.EWError) as e:
        ew.moe_grouped_ffn(x, 1, 128, 2, c, c, c, x, x)
    assert e.value.code == -6


def test_fused_entry_points_empty_batch_and_argument_errors(ew):
    """T = 0 is a no-op (counts zeroed by the permutation call); bad arguments come back as error codes, never as a launch."""
    B = ew.binding
    lib, st = B.lib(), B._stream()
    i32 = dict(dtype=torch.int32, device="cuda")
    H, I, E, N, P, k, S = 256, 128, 8, 1, 12, 2, 1
    counts, offsets = torch.full((P,), 7, **i32), torch.full((P + 1,), 7, **i32)
    emap = torch.arange(E, **i32).repeat(N + 1, 1).contiguous()
    dummy = torch.zeros(4096, dtype=torch.bfloat16, device="cuda")
    ws = B._workspace(max(lib.moe_grouped_ffn_workspace_bytes(1, k + S, H, I, P + S, B.EW_BF16), 256), "cuda")
    assert lib.moe_route_reroute_permute_plan(None, None, emap.data_ptr(), 0, E, k, N, P, 0, None, None, dummy.data_ptr(),
                                              counts.data_ptr(), offsets.data_ptr(), dummy.data_ptr(), None, None, 0, H, I, S,
                                              B.EW_BF16, None, 0, st) == 0
    torch.cuda.synchronize()
    assert int(counts.abs().sum()) == 0 and int(offsets.abs().sum()) == 0
    for fn in (lib.moe_grouped_ffn_planned, lib.moe_grouped_ffn_with_shared):
        assert fn(None, B.EW_BF16, 0, k, H, I, P, S, None, None, None, None, None, None, None, None, None, 0, st) == 0
    assert lib.moe_unpermute_rmsnorm(None, None, None, None, 0, None, 0, k, H, B.EW_BF16, None, 1e-6, None, st) == 0
    # errors: S < 1 for the shared variant, a negative S, H not a multiple of 128, a workspace that is too small
    args = lambda S_, H_, ws_bytes: (dummy.data_ptr(), B.EW_BF16, 1, k, H_, I, P, S_, counts.data_ptr(), offsets.data_ptr(), None,
                                     dummy.data_ptr(), dummy.data_ptr(), dummy.data_ptr(), dummy.data_ptr(), dummy.data_ptr(),
                                     ws.data_ptr(), ws_bytes, st)
    assert lib.moe_grouped_ffn_with_shared(*args(0, H, ws.numel())) == -1          # EW_ERR_INVALID_ARG
    assert lib.moe_grouped_ffn_planned(*args(-1, H, ws.numel())) == -1
    assert lib.moe_grouped_ffn_with_shared(*args(S, 192, ws.numel())) == -6        # EW_ERR_UNSUPPORTED
    assert lib.moe_grouped_ffn_planned(*args(S, H, 256)) == lib.moe_grouped_ffn_with_shared(*args(S, H, 256)) != 0
    assert "workspace" in lib.ew_last_error().decode()
    assert lib.moe_unpermute_rmsnorm(dummy.data_ptr(), counts.data_ptr(), dummy.data_ptr(), None, 0, None, 1, k, H, B.EW_BF16,
                                     dummy.data_ptr(), 1e-6, dummy.data_ptr(), st) == -1   # normed_out must not be out
    torch.cuda.synchronize()


@pytest.mark.parametrize("H,I", [(256, 128), (64, 48), (100, 36), (21, 7), (4, 1)], ids=["c0", "half-tile", "k-tail", "unaligned", "smallest"])
def test_grouped_ffn_f32_tile_edges(ew, H, I):
    """fp32 products at the edges of their 16-feature x 32-row tiles and 16-element steps: row counts around one and two
    row tiles, empty slots between them, contractions that end inside a step, rows without 16-byte alignment."""
    rng = np.random.default_rng(H * 10 + I)
    counts = np.array([0, 1, 15, 16, 17, 0, 31, 32, 33, 64, 65, 200, 0], np.int32)
    P, rows = len(counts), int(counts.sum())
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    por = rng.permutation(rows).astype(np.int32)
    x = rng.standard_normal((rows, H), dtype=np.float32)
    w13 = rng.standard_normal((P, 2 * I, H), dtype=np.float32) * np.float32(0.1)
    w2 = rng.standard_normal((P, H, I), dtype=np.float32) * np.float32(0.1)
    w13[counts == 0], w2[counts == 0] = np.nan, np.nan
    dev = lambda a: torch.from_numpy(a).cuda()
    got = to_f64(ew.moe_grouped_ffn(dev(x), 1, I, P, dev(counts), dev(offsets), dev(por), dev(w13), dev(w2), num_rows=rows))
    for s in np.nonzero(counts)[0]:
        r0, r1 = offsets[s], offsets[s + 1]
        assert rel_l2(got[r0:r1], moe.expert_ffn(x[por[r0:r1]], w13[s], w2[s])) <= 1e-5, f"slot {s}"


@pytest.mark.parametrize("T,k,P,S,H,I", [(1, 1, 3, 0, 256, 256), (2, 6, 16, 2, 2048, 1408), (16, 4, 200, 1, 384, 256), (17, 4, 40, 2, 640, 256),
                                         (32, 3, 9, 0, 256, 384), (33, 2, 12, 2, 1280, 512), (64, 6, 100, 1, 512, 256), (65, 6, 30, 2, 256, 768),
                                         (130, 4, 24, 2, 384, 256), (513, 2, 16, 1, 512, 256), (3, 2, 48, 1, 1280, 512), (3, 4, 12, 0, 1536, 1024),
                                         (16, 4, 20, 1, 1024, 896), (16, 8, 68, 0, 640, 384), (1, 6, 8, 2, 2048, 1408), (16, 4, 23, 1, 1024, 896),
                                         (16, 4, 28, 0, 640, 384), (16, 8, 72, 0, 640, 384),
                                         (129, 2, 9, 1, 256, 384), (160, 1, 5, 1, 512, 256), (161, 3, 7, 1, 256, 128), (300, 2, 24, 2, 256, 256),
                                         (300, 2, 24, 0, 384, 256)])
def test_grouped_ffn_decode_kernel_edges(ew, T, k, P, S, H, I):
    """The kernel of calls with few rows per slot at the edges of its chunks (16, 32, 64, 128 and 160 rows), with contractions
    shorter than its rings, hidden sizes that are an odd multiple of 128, a crowded slot cut into several chunks, more
    workgroups than units (one unit looked up at a time), more units than workgroups whose last round has no room for halves (the
    three before the last four) and, in the last four, units of the first product in halves (of 64 and 128 weight rows): every row
    against the oracle's expert FFN, twice, the same bits both times.
    Weights of deviation 0.02 keep outputs within the range that FFN_MAX_ABS is meant for: a gate or up value has deviation
    0.02 sqrt(2048) = 0.9 at most, an activation about 0.4, an output 0.02 sqrt(1408) 0.4 = 0.3, so below 4 with certainty, where
    bf16 rounds by 2^-7 at most.  At twice the weights outputs are eight times larger and bf16 alone rounds by 2^-5 = 0.03."""
    rng = np.random.default_rng(T * 7 + H)
    ids = np.stack([rng.choice(P, k, replace=False) for _ in range(T)]).astype(np.int32)
    ids[:, 0] = np.where(rng.random(T) < 0.6, 1, ids[:, 0])               # a repeat inside a token is fine here
    flat = ids.reshape(-1)
    por = np.argsort(flat, kind="stable").astype(np.int32)
    counts = np.bincount(flat, minlength=P).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    bf = lambda *shape, scale=1.0: (torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)) * scale).cuda().bfloat16()
    x, w13, w2 = bf(T, H), bf(P, 2 * I, H, scale=0.02), bf(P, H, I, scale=0.02)
    w13[torch.from_numpy(counts == 0).cuda()] = float("nan")
    if S:
        s13, s2 = bf(S, 2 * I, H, scale=0.02), bf(S, H, I, scale=0.02)
        run = lambda: ew.moe_grouped_ffn_with_shared(x, k, I, P, dev(counts), dev(offsets), dev(por), w13, w2, s13, s2)
    else:
        run = lambda: ew.moe_grouped_ffn(x, k, I, P, dev(counts), dev(offsets), dev(por), w13, w2)
    y = run()
    assert torch.equal(y, run())
    got, xs = to_f64(y), to_f64(x)
    for s in np.nonzero(counts)[0]:
        r0, r1 = offsets[s], offsets[s + 1]
        ref = moe.expert_ffn(xs[por[r0:r1] // k], to_f64(w13[s]), to_f64(w2[s]))
        assert rel_l2(got[r0:r1], ref) <= FFN_REL_L2 and max_abs(got[r0:r1], ref) <= FFN_MAX_ABS, f"slot {s}"
    for s in range(S):
        ref = moe.expert_ffn(xs, to_f64(s13[s]), to_f64(s2[s]))
        blk = got[T * k + s * T:T * k + (s + 1) * T]
        assert rel_l2(blk, ref) <= FFN_REL_L2 and max_abs(blk, ref) <= FFN_MAX_ABS, f"shared expert {s}"


@pytest.mark.parametrize("T,k,S,n", [(432, 3, 0, 9), (480, 3, 0, 10), (396, 4, 0, 11), (384, 3, 1, 8), (432, 3, 1, 9)],
                         ids=["one-round", "a-full-round", "more-than-one", "shared-one-round", "shared-more-than-one"])
def test_grouped_ffn_cuts_slots_of_129_to_160_rows_where_one_round_takes_them(ew, T, k, S, n):
    """Slots of 129 to 160 rows, among them slots at the edges, a thin one and idle ones.  Cut at 128 rows where the units of all chunks
    then fit one round of the 256 workgroups (11 and 2 units per chunk here, so 19 chunks), one chunk each where they do not: the plan says which
    (its first word is the number of chunks).  Both give the bits of the kernel whose chunks end at 128, and two slots agree with the oracle."""
    P, H, I = 64, 512, 1408
    rng = np.random.default_rng(T + n)
    rows = np.full(n, 144)
    rows[[0, 1, 2, 3]] = 129, 160, 161, 126                               # 576 rows, as four of 144
    counts = np.zeros(P, np.int32)
    counts[rng.permutation(P - 1)[:n]] = rows
    assert counts.sum() == T * k
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    por = rng.permutation(T * k).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    g = torch.Generator(device="cuda").manual_seed(T)
    bf = lambda *shape, scale=1.0: torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16) * scale
    x, w13, w2 = bf(T, H), bf(P, 2 * I, H, scale=0.02), bf(P, H, I, scale=0.02)
    s13, s2 = (bf(S, 2 * I, H, scale=0.02), bf(S, H, I, scale=0.02)) if S else (None, None)
    args = (x, k, I, P, dev(counts), dev(offsets), dev(por), w13, w2)
    ws = ew.binding._workspace(ew.lib().moe_grouped_ffn_workspace_bytes(T, k + S, H, I, P + S, ew.EW_BF16), "cuda")

    def run(**tune):
        ew.binding.tune_ffn(**tune)
        try:
            y = ew.moe_grouped_ffn_with_shared(*args, s13, s2, ws=ws) if S else ew.moe_grouped_ffn(*args, ws=ws)
        finally:
            ew.binding.tune_ffn()
        return y, int(ws[:4].view(torch.int32))

    y, chunks = run()
    ref, cut = run(path=3, ws_frags=4)
    shared = S * -(-T // 128)
    assert cut == shared + int(sum(-(-c // 128) for c in rows))
    assert chunks == (cut if cut <= 256 // (I // 128 + H // 256) else cut - int(((rows > 128) & (rows <= 160)).sum()))
    assert torch.equal(y, ref)
    got, xs = to_f64(y), to_f64(x)
    for s in (int(np.nonzero(counts == 160)[0][0]), int(np.nonzero(counts == 161)[0][0])):
        r0, r1 = offsets[s], offsets[s + 1]
        want = moe.expert_ffn(xs[por[r0:r1] // k], to_f64(w13[s]), to_f64(w2[s]))
        assert rel_l2(got[r0:r1], want) <= FFN_REL_L2 and max_abs(got[r0:r1], want) <= FFN_MAX_ABS, f"slot {s}"


@pytest.mark.parametrize("frags", [4, 8], ids=["few-rows", "many-rows"])
def test_grouped_ffn_rows_do_not_depend_on_their_place(ew, frags):
    """A token's rows have the same bits wherever it stands in the batch: slots of one to three chunks, crowded and thin ones, and a
    shared expert, whose rows are copies of five tokens in random order.  The same token alone on its slots gives these bits too."""
    T, P, S, H, I = 1100, 8, 1, 640, 384
    rng = np.random.default_rng(frags)
    flat = np.repeat(np.arange(P), [600, 257, 130, 70, 33, 9, 1, 0]).astype(np.int32)[rng.permutation(T)]
    who = rng.integers(0, 5, size=T)
    dev = lambda a: torch.from_numpy(a).cuda()
    bf = lambda *shape, scale=1.0: (torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)) * scale).cuda().bfloat16()
    x5, w13, w2, s13, s2 = bf(5, H), bf(P, 2 * I, H, scale=0.02), bf(P, H, I, scale=0.02), bf(S, 2 * I, H, scale=0.02), bf(S, H, I, scale=0.02)

    def run(who, flat):
        por = np.argsort(flat, kind="stable").astype(np.int32)
        counts = np.bincount(flat, minlength=P).astype(np.int32)
        offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
        ew.binding.tune_ffn(path=3, ws_frags=frags)
        try:
            y = ew.moe_grouped_ffn_with_shared(x5[dev(who)].contiguous(), 1, I, P, dev(counts), dev(offsets), dev(por), w13, w2, s13, s2)
        finally:
            ew.binding.tune_ffn()
        n = len(flat)
        return y[:n].view(torch.int16).cpu().numpy(), y[n:].view(torch.int16).cpu().numpy(), flat[por], who[por]

    y, sh, slot, tok = run(who, flat)
    y1, sh1, slot1, tok1 = run(np.arange(5 * P) % 5, (np.arange(5 * P) // 5).astype(np.int32))    # every token once on every slot
    for r in range(5 * P):
        rows = y[(slot == slot1[r]) & (tok == tok1[r])]
        assert (rows == y1[r]).all(), f"slot {slot1[r]}, token {tok1[r]}: {int((rows != y1[r]).any(axis=1).sum())} of {len(rows)} rows differ"
    for t in range(5):
        assert (sh[who == t] == sh1[t]).all(), f"shared expert, token {t}"


@pytest.mark.parametrize("T,k,P,S,H,I,used", [(768, 2, 64, 1, 384, 256, 64), (768, 2, 64, 1, 384, 256, 6), (1100, 4, 96, 0, 256, 128, 96),
                                              (1100, 4, 96, 0, 256, 128, 4), (520, 2, 2046, 2, 128, 128, 5)],
                         ids=["spread", "few-used", "spread-no-shared", "four-used", "largest-pool"])
def test_grouped_ffn_counts_choose_the_kernel(ew, T, k, P, S, H, I, used):
    """More than 512 tokens on more slots than they need: the counts decide on the device which kernel runs, by the average
    rows of the slots in use.  Traffic over all slots and over a few of them, both against the oracle and against each
    kernel asked for by name, bit for bit with the one the rule names."""
    rng = np.random.default_rng(T + used)
    slots = np.sort(rng.choice(P, used, replace=False))
    ids = slots[np.stack([rng.choice(used, k, replace=False) for _ in range(T)])].astype(np.int32)
    flat = ids.reshape(-1)
    por = np.argsort(flat, kind="stable").astype(np.int32)
    counts = np.bincount(flat, minlength=P).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    bf = lambda *shape, scale=1.0: (torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)) * scale).cuda().bfloat16()
    x, w13, w2 = bf(T, H), bf(P, 2 * I, H, scale=0.02), bf(P, H, I, scale=0.02)
    s13, s2 = (bf(S, 2 * I, H, scale=0.02), bf(S, H, I, scale=0.02)) if S else (None, None)
    args = (dev(counts), dev(offsets), dev(por), w13, w2)

    def run(frags=0):
        ew.binding.tune_ffn(path=3 if frags else 0, ws_frags=frags)
        try:
            return ew.moe_grouped_ffn_with_shared(x, k, I, P, *args, s13, s2) if S else ew.moe_grouped_ffn(x, k, I, P, *args)
        finally:
            ew.binding.tune_ffn()

    y = run()
    few, many = run(4), run(8)
    active = int((counts > 0).sum()) + S
    assert not torch.equal(few, many)                                      # their sums differ in order: the next line tells them apart
    assert torch.equal(y, many if T * (k + S) > 128 * active else few)
    xs = to_f64(x)
    for got in (to_f64(few), to_f64(many)):
        for s in np.nonzero(counts)[0][:12]:
            r0, r1 = offsets[s], offsets[s + 1]
            ref = moe.expert_ffn(xs[por[r0:r1] // k], to_f64(w13[s]), to_f64(w2[s]))
            assert rel_l2(got[r0:r1], ref) <= FFN_REL_L2 and max_abs(got[r0:r1], ref) <= FFN_MAX_ABS, f"slot {s}"
        for s in range(S):
            blk = got[T * k + s * T:T * k + (s + 1) * T]
            assert rel_l2(blk, moe.expert_ffn(xs, to_f64(s13[s]), to_f64(s2[s]))) <= FFN_REL_L2, f"shared expert {s}"


@pytest.mark.parametrize("T,E,k,N,e_max,S,H,I,renorm,repeat", [
    (1, 64, 6, 4, 16, 2, 256, 128, False, False),       # a token's pairs alone
    (4, 8, 2, 2, 2, 0, 128, 128, True, False),          # one selecting wave, one expert per lane
    (13, 96, 4, 20, 16, 1, 256, 128, True, False),      # a ragged wave, eight experts per lane
    (16, 256, 16, 1, 8, 3, 128, 128, False, False),     # sixteen experts per lane, as many choices as lanes
    (17, 16, 5, 3, 4, 2, 128, 256, True, False),        # chunks of 32 rows
    (32, 24, 16, 2, 16, 16, 128, 128, False, False),    # most pairs, most shared chunks
    (33, 64, 6, 4, 16, 2, 256, 128, False, False),      # chunks of 64 rows, the ninth of the selecting waves with one token
    (61, 128, 8, 124, 15, 1, 128, 128, True, False),    # the last selecting wave ragged, 1988 slots
    (64, 64, 8, 0, 1, 0, 128, 128, False, False),       # most tokens, most pairs, no adapters
    (64, 64, 1, 5, 16, 2, 128, 128, False, False),
    (20, 8, 6, 2, 4, 2, 256, 128, False, True),         # a map that sends two experts to one slot: slots with more rows than tokens
    (64, 8, 8, 1, 4, 1, 128, 128, True, True),
])
def test_layer_that_routes_itself_equals_the_separate_launches(ew, T, E, k, N, e_max, S, H, I, renorm, repeat):
    """A pass of few tokens routes inside the FFN's launch; with its logits given it runs permutation and FFN as launches of their
    own.  Everything the two leave behind has the same bits, on three passes in a row over other tokens (the counters are zeroed
    again every time), and slots that no token visits are not read."""
    from types import SimpleNamespace
    from paper_2508_17624_amd.layer import MoELayer
    rng = np.random.default_rng([T, E, k, N])
    g = torch.Generator(device="cuda").manual_seed(T + 100 * E)
    bf = lambda *shape, scale=1.0: (torch.randn(shape, generator=g, device="cuda") * scale).bfloat16()
    P = E + N * e_max
    emap = np.tile(np.arange(E, dtype=np.int32), (N + 1, 1))
    for a in range(1, N + 1):
        ids = np.sort(rng.choice(E, size=min(E, e_max), replace=False))
        emap[a, ids] = E + (a - 1) * e_max + np.arange(len(ids))
    if repeat:
        emap //= 2
    w13, w2 = bf(P, 2 * I, H, scale=0.05), bf(P, H, I, scale=0.05)
    backed = torch.zeros(P, dtype=torch.bool)
    backed[torch.from_numpy(np.unique(emap)).long()] = True
    w13[~backed.cuda()] = float("nan")
    w2[~backed.cuda()] = float("nan")
    emap_t = torch.from_numpy(emap).cuda()
    pool = SimpleNamespace(M=E, N=N, P=P, view=lambda l: (w13.data_ptr(), w2.data_ptr(), emap_t.data_ptr(), P))
    shared = (bf(S, 2 * I, H, scale=0.05), bf(S, H, I, scale=0.05)) if S else (None, None)
    Wg = torch.randn((E, H), generator=g, device="cuda") * 0.1
    # (the adapters' gate bias, in every second case: such a pass has its scores from the same launch)
    bias = torch.randn((N + 1, E), generator=g, device="cuda") if T % 2 == 0 else None
    make = lambda: MoELayer(pool, 0, Wg, shared[0], shared[1], k, I, T, torch.bfloat16, bias=bias, renormalize=renorm)
    fused, apart = make(), make()
    names = ("ids", "w", "slot", "counts", "offsets", "por", "rop", "y", "y_shared")
    first_word = lambda layer: int(layer.ws_ffn[:4].view(torch.int32))          # of the plan: its size, which no pass that routes itself writes
    for b in (fused.buf, apart.buf):
        b.ws_ffn.fill_(0x5A)                                                    # whatever a workspace holds before its first call
    for turn in range(3):
        x, aid = bf(T, H), torch.from_numpy(rng.integers(0, N + 1, T).astype(np.int32)).cuda()
        last = dict(residual=bf(T, H), eps=1e-6) if turn else {}                # (a residual and the next layer's norm, as in a stack)
        norms = [torch.empty_like(x) if turn else None for _ in range(2)]
        got = fused.forward(x, aid, normed_out=norms[0], **last).clone()
        want = apart.forward(x, aid, fused.logits[:T].clone(), normed_out=norms[1], **last).clone()
        assert first_word(fused) == 0x5A5A5A5A and 0 < first_word(apart) <= T * k + S * T, "which of the two ways the passes took"
        torch.testing.assert_close(fused.logits, ew.moe_gate_logits(x, Wg, None if bias is None else aid, bias), rtol=0, atol=0)
        assert not turn or (torch.equal(*norms) and torch.isfinite(norms[0].float()).all()), f"pass {turn}: norm"
        for name in names:
            assert torch.equal(getattr(fused, name), getattr(apart, name)), f"pass {turn}: {name}"
        assert torch.equal(got, want) and torch.isfinite(got.float()).all(), f"pass {turn}"



def test_what_keeps_a_pass_from_routing_itself_is_reported(ew):
    """Arguments that a pass of few tokens cannot route itself with take the separate calls, which refuse them with their own
    message: the same one as for a pass whose logits are given.  Nothing is left behind that the next pass would see."""
    import ctypes
    from types import SimpleNamespace
    from paper_2508_17624_amd.layer import MoELayer
    B = ew.binding
    T, E, k, N, P, S, H, I = 20, 16, 2, 1, 24, 1, 128, 128
    g = torch.Generator(device="cuda").manual_seed(5)
    bf = lambda *shape, scale=1.0: (torch.randn(shape, generator=g, device="cuda") * scale).bfloat16()
    w13, w2, emap = bf(P, 2 * I, H, scale=0.05), bf(P, H, I, scale=0.05), torch.arange(E, dtype=torch.int32, device="cuda").repeat(N + 1, 1)
    pool = SimpleNamespace(M=E, N=N, P=P, view=lambda l: (w13.data_ptr(), w2.data_ptr(), emap.data_ptr(), P))
    layer = MoELayer(pool, 0, torch.randn((E, H), generator=g, device="cuda"), bf(S, 2 * I, H, scale=0.05), bf(S, H, I, scale=0.05), k, I, T, torch.bfloat16)
    x, aid = bf(T, H), torch.zeros(T, dtype=torch.int32, device="cuda")
    want = layer.forward(x, aid).clone()
    given = layer.logits.clone()

    def call(scores, adapter=aid, **broken):
        layer._current()
        d = B.LayerDesc.from_buffer_copy(layer._desc)
        for name, v in broken.items():
            setattr(d, name, v)
        rc = B.lib().moe_layer_forward(ctypes.byref(d), x.data_ptr(), None if adapter is None else adapter.data_ptr(), T,
                                       None if scores is None else scores.data_ptr(), None, layer.out.data_ptr(), None, 0.0, B._stream())
        return rc, B.lib().ew_last_error().decode() if rc else ""

    layer._current()
    d = layer._desc
    cases = [{n: None} for n in ("expert_map", "w13", "w2", "w13_shared", "w2_shared", "ids", "w", "slot", "counts", "offsets", "pair_of_row",
                                 "row_of_pair", "y", "ws_perm", "ws_ffn")]
    cases += [dict(ws_ffn=d.ws_ffn + 128), dict(ws_ffn_bytes=d.ws_ffn_bytes - 256), dict(ws_perm=d.ws_perm + 128), dict(ws_perm_bytes=1),
              dict(k=E + 1), dict(N=-1), dict(P=4096), dict(I=192), dict(adapter=None)]
    for broken in cases:
        rc, why = call(None, **broken)
        assert rc < 0 and (rc, why) == call(given, **broken), f"{broken}: {rc} {why}"
        assert call(None) == (0, "") and torch.equal(layer.out[:T], want), f"the pass after {broken}"
    for name in ("Wg", "logits"):
        assert call(None, **{name: None})[0] == -1 and call(given, **{name: None}) == (0, ""), name
