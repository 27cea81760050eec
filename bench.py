#!/usr/bin/env python3
"""Benchmark of the ExpertWeave MoE-layer hot path on one MI355X.

A step is one pass of the whole hot path over one batch of synthetic input already resident in
HBM: router scores -> fused top-k + rerouting + permutation -> grouped SwiGLU FFN over the VMM
expert pool -> shared experts -> weighted un-permute.  The headline workload is configuration 2
(DeepSeek-V2-Lite-shaped layer, 8192-token prefill, 20 adapters); the decode configuration 1 and
the base-only comparison are reported in `extras` of the same JSON line.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu-baseline] [--no-extras]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import numpy as np
import torch

import workloads as wl

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, published
MFMA_BF16_PEAK_TFLOPS = 2500.0  # MI355X dense bf16, published
# HBM bytes (read + written) of one launch sequence cannot be read live: they come from rocprofv3 FETCH_SIZE / WRITE_SIZE
# runs scaled by a plain copy of known size.  The figure is taken from the committed summary of those runs (the line
# "traffic_bytes_per_call = ..." of the profile that covers the workload), so it changes only when the profile is regenerated.
PROFILE_OF = {"c2_dsv2lite_prefill": "grouped_ffn_c2_prefill_20adapters.md", "c1_dsv2lite_decode": "grouped_ffn_c1_decode.md",
              "c3_reroute_permute_int": "reroute_permute_c3.md"}


def traffic_bytes(workload):
    import re
    try:
        text = open(os.path.join(ROOT, "profiles", PROFILE_OF[workload])).read()
    except (KeyError, OSError):
        return None
    m = re.search(r"traffic_bytes_per_call\s*=\s*([0-9.eE+]+)", text)
    return float(m.group(1)) if m else None


def dev(a: np.ndarray) -> torch.Tensor:
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).cuda()
    return torch.from_numpy(a).cuda()


class LayerSetup:
    """One configuration loaded on the GPU: VMM pool, layer object, resident inputs."""

    def __init__(self, cfg, ew, layer_mod):
        self.cfg = cfg
        t0 = time.time()
        tuned = wl.tuned_sets(cfg)
        el = 2
        self.pool = ew.ExpertPool(1, cfg.M, cfg.N, cfg.E_max, 2 * cfg.I * cfg.H * el, cfg.H * cfg.I * el)
        host = lambda a: torch.from_numpy(a.view(np.int16))
        b13, b2 = wl.stacked_expert_weights(cfg, 0, 0, cfg.M)
        self.pool.map(0, 0, list(range(cfg.M)), host(b13), host(b2))
        del b13, b2
        for a in range(cfg.N):
            a13, a2 = wl.stacked_expert_weights(cfg, 0, a + 1, len(tuned[a]))
            self.pool.map(0, a + 1, [int(e) for e in tuned[a]], host(a13), host(a2))
        sh13, sh2 = wl.shared_weights(cfg)
        self.tuned = tuned
        self.x = dev(wl.tokens(cfg))
        self.aid = dev(wl.adapter_ids(cfg))
        self.aid0 = torch.zeros_like(self.aid)
        bias = dev(wl.logit_bias_table(cfg, tuned)) if cfg.gate_bias else None
        self.layer = layer_mod.MoELayer(self.pool, 0, dev(wl.gate_weight(cfg)), dev(sh13), dev(sh2), cfg.k, cfg.I, cfg.T,
                                        torch.bfloat16, bias=bias)
        torch.cuda.synchronize()
        self.setup_s = time.time() - t0

    def step(self, aid=None):
        return self.layer.forward(self.x, self.aid if aid is None else aid)

    def time_steps(self, steps, warmup, aid=None):
        """(wall-clock mean, median of per-step event pairs) in seconds over exactly `steps` steps."""
        return timed_steps(lambda: self.step(aid), steps, warmup)

    def ffn_call(self, B):
        """The layer's grouped-FFN call as its step makes it (routed and shared experts in one call), minus the plan
        hand-over from the permutation call: the call builds its own plan here."""
        L, cfg = self.layer, self.cfg
        lib, st, b = B.lib(), B._stream(), self.layer.buf
        if cfg.S:
            return lambda: B._check(lib.moe_grouped_ffn_with_shared(
                self.x.data_ptr(), L.dt, cfg.T, cfg.k, cfg.H, cfg.I, cfg.P, cfg.S, b.counts.data_ptr(), b.offsets.data_ptr(),
                b.por.data_ptr(), L.w13_base, L.w2_base, L.shared_w13.data_ptr(), L.shared_w2.data_ptr(), b.y.data_ptr(),
                b.ws_ffn.data_ptr(), b.ws_ffn.numel(), st))
        return lambda: B._check(lib.moe_grouped_ffn(
            self.x.data_ptr(), L.dt, cfg.T, cfg.k, cfg.H, cfg.I, cfg.P, b.counts.data_ptr(), b.offsets.data_ptr(),
            b.por.data_ptr(), L.w13_base, L.w2_base, b.y.data_ptr(), b.ws_ffn.data_ptr(), b.ws_ffn.numel(), st))

    def ffn_work(self, active):
        """(flop, weight bytes) of that call: every sorted row through one expert, every active expert's weights once."""
        cfg = self.cfg
        return cfg.T * (cfg.k + cfg.S) * 6.0 * cfg.H * cfg.I, (active + cfg.S) * 3.0 * cfg.H * cfg.I * 2

    def time_ffn_cold(self, B, flush, iters=10):
        """The grouped-FFN call with cold caches: a large streaming read evicts L2 and the memory-side cache first."""
        call = self.ffn_call(B)
        ms = []
        for _ in range(iters):
            flush()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            call()
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        ms.sort()
        return ms[len(ms) // 2] / 1e3

    def time_ffn(self, steps, B):
        """Average and median duration of the grouped-FFN call alone (HIP events on the launch stream)."""
        call = self.ffn_call(B)
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
        for i in range(steps + 3):
            if i >= 3:
                ev[i - 3][0].record()
            call()
            if i >= 3:
                ev[i - 3][1].record()
        torch.cuda.synchronize()
        ms = sorted(a.elapsed_time(b) for a, b in ev)
        return sum(ms) / len(ms) / 1e3, ms[len(ms) // 2] / 1e3

    def active_slots(self):
        return int((self.layer.counts > 0).sum().item())

    def stage_us(self, B, iters=30):
        """Median microseconds of each call of a layer step on its own (HIP events around the single call, so every
        figure carries one launch gap; the step itself runs them back to back)."""
        L, cfg = self.layer, self.cfg
        lib, st, b = B.lib(), B._stream(), self.layer.buf
        T, k, H, I, P = cfg.T, cfg.k, cfg.H, cfg.I, cfg.P
        bias_ptr = L.bias.data_ptr() if L.bias is not None else None
        gate = lambda: B._check(lib.moe_gate_logits(self.x.data_ptr(), L.dt, L.Wg.data_ptr(), T, H, cfg.M,
                                                    self.aid.data_ptr() if bias_ptr else None, bias_ptr, b.logits.data_ptr(), st))
        route = lambda: L.route(self.x, self.aid, logits=b.logits, plan=True)
        S = cfg.S
        sh_ptr = b.y.data_ptr() + T * k * H * 2 if S else None
        comb = lambda: B._check(lib.moe_unpermute(b.y.data_ptr(), b.rop.data_ptr(), b.w.data_ptr(), sh_ptr, S, None, T, k, H, L.dt,
                                                  b.out.data_ptr(), st))
        self.step()
        out = {}
        for name, fn in (("gate_logits", gate), ("topk_reroute_permute_plan", route), ("grouped_ffn", self.ffn_call(B)),
                         ("unpermute", comb)):
            out[name] = time_call(fn, iters=iters)[0] * 1e6
        return out


def timed_steps(step, steps, warmup):
    """Runs `warmup` untimed steps, then exactly `steps` steps between two device synchronisations.  Returns the
    wall-clock mean per step and the median over the steps of HIP-event pairs recorded around each one (seconds)."""
    for _ in range(warmup):
        step()
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for a, b in ev:
        a.record(); step(); b.record()
    torch.cuda.synchronize()
    wall = (time.perf_counter() - t0) / steps
    ms = sorted(a.elapsed_time(b) for a, b in ev)
    return wall, ms[len(ms) // 2] / 1e3


def measured_peaks(B, lib):
    """What this GPU sustains, measured in this run with the library's probe kernels: a 1 GiB streaming read and copy
    (HBM) and a register-resident loop of the FFN's bf16 matrix-core instruction with constant and with random operands
    (the chip lowers its clock under the load of random data)."""
    st = B._stream()
    n = 1 << 30
    src = torch.empty(n, dtype=torch.uint8, device="cuda").random_(0, 255)
    dst = torch.empty(n, dtype=torch.uint8, device="cuda")
    out = {}
    t, _ = time_call(lambda: B._check(lib.ew_probe_stream(src.data_ptr(), dst.data_ptr(), n, 1, st)), iters=10)
    out["hbm_read_GBs"] = n / t / 1e9
    t, _ = time_call(lambda: B._check(lib.ew_probe_stream(src.data_ptr(), dst.data_ptr(), n, 0, st)), iters=10)
    out["hbm_copy_GBs_read_plus_written"] = 2 * n / t / 1e9
    del src, dst
    wgs, iters = 256 * 4, 4000
    buf = torch.zeros(4 * wgs, dtype=torch.int64, device="cuda")
    flop = wgs * 8 * iters * 8 * 32768.0
    for name, rnd in (("constant", 0), ("random", 1)):
        t, _ = time_call(lambda: B._check(lib.ew_probe_mfma_bf16(wgs, iters, rnd, buf.data_ptr(), st)), iters=10)
        ticks = buf.view(wgs, 4)[:, :2].double().cpu().numpy()
        out[f"mfma_bf16_{name}_operands_TFLOPs"] = flop / t / 1e12
        out[f"shader_clock_GHz_{name}_operands"] = float((ticks[:, 0] / ticks[:, 1]).mean() * 0.1)
    out["note"] = ("ew_probe_stream over 1 GiB and ew_probe_mfma_bf16 (1024 workgroups of 8 waves, 4000 x 8 "
                   "v_mfma_f32_32x32x16_bf16 per wave), medians of 10 launches timed with HIP events in this run")
    return out


def time_call(fn, iters=30, warm=3):
    """Median and mean seconds of fn() over `iters` calls, HIP events on the current stream."""
    for _ in range(warm):
        fn()
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(iters)]
    for a, b in ev:
        a.record(); fn(); b.record()
    torch.cuda.synchronize()
    ms = sorted(a.elapsed_time(b) for a, b in ev)
    return ms[len(ms) // 2] / 1e3, sum(ms) / len(ms) / 1e3


def layer_ablation(B, lib, s, t_step):
    """Inside one layer: fused top-k + rerouting + permutation against router top-k, the three single rerouting
    operators and the permutation as separate launches."""
    st = B._stream()
    i32 = dict(dtype=torch.int32, device="cuda")
    L, cfg = s.layer, s.cfg
    T, k, P, N, E = cfg.T, cfg.k, cfg.P, cfg.N, cfg.M
    b = L.buf
    ws_so = B._workspace(lib.moe_reroute_singleop_workspace_bytes(T, k), "cuda")
    ident, zero = torch.arange(P, **i32).reshape(1, P).contiguous(), torch.zeros(T, **i32)
    slot_tmp = torch.empty((T, k), **i32)
    L.route(s.x, s.aid)

    def fused():
        B._check(lib.moe_route_reroute_permute(b.logits.data_ptr(), s.aid.data_ptr(), L.emap, T, E, k, N, P, 0, b.ids.data_ptr(),
                                               b.w.data_ptr(), b.slot.data_ptr(), b.counts.data_ptr(), b.offsets.data_ptr(),
                                               b.por.data_ptr(), b.rop.data_ptr(), B._ptr(b.ws_perm),
                                               b.ws_perm.numel() if b.ws_perm is not None else 0, st))

    def unfused():
        B._check(lib.moe_route_topk(b.logits.data_ptr(), T, E, k, 0, b.ids.data_ptr(), b.w.data_ptr(), st))
        B._check(lib.moe_reroute_singleop(b.ids.data_ptr(), s.aid.data_ptr(), L.emap, T, k, E, N, slot_tmp.data_ptr(),
                                          ws_so.data_ptr(), ws_so.numel(), st))
        B._check(lib.moe_reroute_permute(slot_tmp.data_ptr(), zero.data_ptr(), ident.data_ptr(), T, k, P, 0, P,
                                         b.slot.data_ptr(), b.counts.data_ptr(), b.offsets.data_ptr(), b.por.data_ptr(),
                                         b.rop.data_ptr(), B._ptr(b.ws_perm), b.ws_perm.numel() if b.ws_perm is not None else 0, st))

    tf, _ = time_call(fused)
    tu, _ = time_call(unfused)
    fused()
    return {"workload": cfg.name, "fused_topk_reroute_permute_us": tf * 1e6, "topk_singleop_permute_us": tu * 1e6,
            "fused_pct_of_layer_step": tf / t_step * 100.0, "unfused_pct_of_layer_step": tu / t_step * 100.0,
            "layer_overhead_if_unfused_pct": (tu - tf) / t_step * 100.0}


def second_workload_sweep(s2, steps=10):
    """Chunked-prefill sizes and skewed adapter popularity on the configuration-2 layer (the axes of the paper's
    Fig. 5 restricted to the MoE layer): T in {512, 2048}, n adapters in {5, 10, 20} drawn with the power-law shape
    alpha in {1, 0.3, 0.1}; latency of one layer step, active slots, and the same T with base-only traffic."""
    rows = []
    cfg = s2.cfg
    for T in (512, 2048):
        x = s2.x[:T]
        t_base, _ = time_call(lambda: s2.layer.forward(x, s2.aid0[:T]), iters=steps)
        for n in (5, 10, 20):
            for alpha in (1.0, 0.3, 0.1):
                aid = dev(wl.adapter_ids_powerlaw(cfg, T, n, alpha))
                t, _ = time_call(lambda: s2.layer.forward(x, aid), iters=steps)
                active = int((s2.layer.counts > 0).sum().item())
                rows.append({"T": T, "adapters": n, "alpha": alpha, "ms": t * 1e3, "tokens_per_s": T / t,
                             "active_slots": active, "base_only_ms": t_base * 1e3, "overhead_pct": (t / t_base - 1.0) * 100.0})
    return rows


def c3_pool(c3):
    """The expert map of the integer microbenchmark, written by expert_pool_map into a pool whose experts are one
    256-byte placeholder each (the configuration has no weights); returns (pool, device pointer of the map)."""
    import paper_2508_17624_amd as ew
    pool = ew.ExpertPool(1, c3.M, c3.N, c3.E_max, 256, 256)
    pool.map(0, 0, list(range(c3.M)))
    for a, J in enumerate(wl.tuned_sets(c3), start=1):
        pool.map(0, a, [int(e) for e in J])
    torch.cuda.synchronize()
    return pool, pool.view(0)[2]


def ablation_rerouting(B, lib, s2, t_step_c2, s1=None, t_step_c1=None):
    """Fused versus unfused rerouting (the analogue of the paper's Sec. 5.3 / Fig. 7 comparison), on the integer
    microbenchmark (configuration 3) and inside the configuration-2 layer.  All buffers are preallocated."""
    out = {}
    st = B._stream()
    i32 = dict(dtype=torch.int32, device="cuda")
    # --- configuration 3: T = 2^20 tokens x top-6, integer only
    c3 = wl.get_config(3)
    T, k, P, N, E = c3.T, c3.k, c3.P, c3.N, c3.M
    pool3, emap_ptr = c3_pool(c3)
    ids, aid = dev(wl.distinct_topk_ids(c3)), dev(wl.adapter_ids(c3))
    slot, counts, offsets = torch.empty((T, k), **i32), torch.empty(P, **i32), torch.empty(P + 1, **i32)
    por, rop = torch.empty(T * k, **i32), torch.empty(T * k, **i32)
    ws = B._workspace(lib.moe_reroute_permute_workspace_bytes(T, k, P), "cuda")
    ws_so = B._workspace(lib.moe_reroute_singleop_workspace_bytes(T, k), "cuda")
    ident, zero = torch.arange(P, **i32).reshape(1, P).contiguous(), torch.zeros(T, **i32)
    slot2 = torch.empty((T, k), **i32)

    def fused():
        B._check(lib.moe_reroute_permute(ids.data_ptr(), aid.data_ptr(), emap_ptr, T, k, E, N, P, slot.data_ptr(),
                                         counts.data_ptr(), offsets.data_ptr(), por.data_ptr(), rop.data_ptr(), ws.data_ptr(),
                                         ws.numel(), st))

    def unfused():
        B._check(lib.moe_reroute_singleop(ids.data_ptr(), aid.data_ptr(), emap_ptr, T, k, E, N, slot2.data_ptr(),
                                          ws_so.data_ptr(), ws_so.numel(), st))
        B._check(lib.moe_reroute_permute(slot2.data_ptr(), zero.data_ptr(), ident.data_ptr(), T, k, P, 0, P, slot.data_ptr(),
                                         counts.data_ptr(), offsets.data_ptr(), por.data_ptr(), rop.data_ptr(), ws.data_ptr(),
                                         ws.numel(), st))

    tf, _ = time_call(fused)
    tu, _ = time_call(unfused)
    alg = T * 100.0                                      # bytes: 28 read + 72 written per token at k = 6
    out["c3_reroute_permute"] = {"workload": c3.name, "tokens": T, "fused_us": tf * 1e6, "unfused_us": tu * 1e6,
                                 "unfused_over_fused": tu / tf,
                                 "roofline": {"bound": "hbm", "kernel": "moe_reroute_permute (k_hist + k_colscan + k_scatter_tok)",
                                              "achieved": alg / tf / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                                              "frac": alg / tf / 1e9 / HBM_PEAK_GBS, "traffic": traffic_bytes(c3.name),
                                              "algorithmic_bytes": alg}}
    pool3.close()
    out["c2_layer"] = layer_ablation(B, lib, s2, t_step_c2)
    if s1 is not None:
        out["c1_layer"] = layer_ablation(B, lib, s1, t_step_c1)
    return out


def pool_modes(B, lib, ew, layer_mod, cfg, steps):
    """The same routed FFN call on (i) the VMM pool (pages only under loaded experts), (ii) the padded pool (every slot
    backed, Sec. 3.1) and (iii) one plain device allocation: the analogue of the paper's virtual-tensor-versus-padding
    comparison (Sec. 5.3) plus the memory each mode holds."""
    out = {}
    el = 2
    tuned = wl.tuned_sets(cfg)
    host = lambda a: torch.from_numpy(a.view(np.int16))
    base = wl.stacked_expert_weights(cfg, 0, 0, cfg.M)
    adapters = [wl.stacked_expert_weights(cfg, 0, a + 1, len(tuned[a])) for a in range(cfg.N)]
    sh13, sh2 = wl.shared_weights(cfg)
    x, aid = dev(wl.tokens(cfg)), dev(wl.adapter_ids(cfg))
    bias = dev(wl.logit_bias_table(cfg, tuned)) if cfg.gate_bias else None
    Wg = dev(wl.gate_weight(cfg))
    for mode, flags in (("vmm", ew.EW_POOL_VMM), ("padded", ew.EW_POOL_PADDED)):
        pool = ew.ExpertPool(1, cfg.M, cfg.N, cfg.E_max, 2 * cfg.I * cfg.H * el, cfg.H * cfg.I * el, flags=flags)
        layer_mod.load_layer(pool, 0, (host(base[0]), host(base[1])), [(host(a), host(b)) for a, b in adapters], tuned)
        layer = layer_mod.MoELayer(pool, 0, Wg, dev(sh13), dev(sh2), cfg.k, cfg.I, cfg.T, torch.bfloat16, bias=bias)
        layer.route(x, aid)
        b, st = layer.buf, B._stream()
        fn = lambda: B._check(lib.moe_grouped_ffn(x.data_ptr(), layer.dt, cfg.T, cfg.k, cfg.H, cfg.I, cfg.P, b.counts.data_ptr(),
                                                  b.offsets.data_ptr(), b.por.data_ptr(), layer.w13_base, layer.w2_base,
                                                  b.y.data_ptr(), b.ws_ffn.data_ptr(), b.ws_ffn.numel(), st))
        med, _ = time_call(fn, iters=steps)
        stt = pool.stats()
        out[mode] = {"routed_ffn_us": med * 1e6, "bytes_physical": stt["pages_mapped"] * stt["page_bytes"],
                     "bytes_virtual": stt["bytes_virtual"], "bytes_experts": stt["bytes_experts"]}
        if mode == "vmm":
            counts, offsets, por = b.counts.clone(), b.offsets.clone(), b.por.clone()
        del layer
        pool.close()
    # (iii) plain allocation holding all P slots (what a framework tensor would be)
    w13 = torch.empty((cfg.P, 2 * cfg.I, cfg.H), dtype=torch.bfloat16, device="cuda")
    w2 = torch.empty((cfg.P, cfg.H, cfg.I), dtype=torch.bfloat16, device="cuda")
    w13[:cfg.M].copy_(dev(base[0])); w2[:cfg.M].copy_(dev(base[1]))
    for a, (a13, a2) in enumerate(adapters):
        if len(a13):
            s0 = cfg.M + a * cfg.E_max
            w13[s0:s0 + len(a13)].copy_(dev(a13)); w2[s0:s0 + len(a2)].copy_(dev(a2))
    y = torch.empty((cfg.T * cfg.k, cfg.H), dtype=torch.bfloat16, device="cuda")
    ws = B._workspace(lib.moe_grouped_ffn_workspace_bytes(cfg.T, cfg.k, cfg.H, cfg.I, cfg.P, B.EW_BF16), "cuda")
    st = B._stream()
    fn = lambda: B._check(lib.moe_grouped_ffn(x.data_ptr(), B.EW_BF16, cfg.T, cfg.k, cfg.H, cfg.I, cfg.P, counts.data_ptr(),
                                              offsets.data_ptr(), por.data_ptr(), w13.data_ptr(), w2.data_ptr(), y.data_ptr(),
                                              ws.data_ptr(), ws.numel(), st))
    med, _ = time_call(fn, iters=steps)
    out["plain_allocation"] = {"routed_ffn_us": med * 1e6, "bytes_physical": (w13.numel() + w2.numel()) * 2}
    out["vmm_vs_padded_pct"] = (out["vmm"]["routed_ffn_us"] / out["padded"]["routed_ffn_us"] - 1.0) * 100.0
    out["vmm_vs_plain_pct"] = (out["vmm"]["routed_ffn_us"] / out["plain_allocation"]["routed_ffn_us"] - 1.0) * 100.0
    out["memory_saved_vs_padded_pct"] = (1.0 - out["vmm"]["bytes_physical"] / out["padded"]["bytes_physical"]) * 100.0
    return out


def adapter_churn(ew, cfg, flags, rounds=6):
    """Evict one adapter of one layer and load it again (Sec. 4.2 load / unload): wall-clock per call.  With the
    default lazy eviction the pages stay parked in place and come back without a VMM call; with EW_POOL_EAGER_UNMAP
    they are unmapped at eviction and mapped again from the free list."""
    el = 2
    tuned = wl.tuned_sets(cfg)
    pool = ew.ExpertPool(1, cfg.M, cfg.N, cfg.E_max, 2 * cfg.I * cfg.H * el, cfg.H * cfg.I * el, flags=flags)
    host = lambda a: torch.from_numpy(a.view(np.int16)).pin_memory()
    b13, b2 = wl.stacked_expert_weights(cfg, 0, 0, cfg.M)
    pool.map(0, 0, list(range(cfg.M)), torch.from_numpy(b13.view(np.int16)), torch.from_numpy(b2.view(np.int16)))
    a = 1
    J = [int(e) for e in tuned[a - 1]]
    a13, a2 = wl.stacked_expert_weights(cfg, 0, a, len(J))
    h13, h2 = host(a13), host(a2)
    t_map, t_unmap = [], []
    for r in range(rounds):
        t0 = time.perf_counter(); pool.map(0, a, J, h13, h2); torch.cuda.synchronize(); t_map.append(time.perf_counter() - t0)
        t0 = time.perf_counter(); pool.unmap(0, a); torch.cuda.synchronize(); t_unmap.append(time.perf_counter() - t0)
    st = pool.stats()
    nbytes = len(J) * 3 * cfg.H * cfg.I * el
    pool.close()
    first, rest = t_map[0], sorted(t_map[1:])[len(t_map[1:]) // 2]
    return {"experts": len(J), "bytes": nbytes, "map_first_ms": first * 1e3, "map_reusing_pages_ms": rest * 1e3,
            "unmap_ms": sorted(t_unmap)[len(t_unmap) // 2] * 1e3, "host_to_device_GBs_reusing_pages": nbytes / rest / 1e9,
            "pages_created": st["pages_created"], "pages_free_after": st["pages_free"], "pages_parked_after": st["pages_parked"]}


class StackSetup:
    """Configuration 4: L stacked layers over one VMM pool, one decode step through all of them."""

    def __init__(self, cfg, ew, layer_mod):
        self.cfg = cfg
        t0 = time.time()
        L = cfg.L
        self.pool = ew.ExpertPool(L, cfg.M, cfg.N, cfg.E_max, 2 * cfg.I * cfg.H * 2, cfg.H * cfg.I * 2)
        host = lambda a: torch.from_numpy(a.view(np.int16))
        gates, shared = [], []
        for l in range(L):
            tuned = wl.tuned_sets(cfg, l)
            b13, b2 = wl.stacked_expert_weights(cfg, l, 0, cfg.M)
            self.pool.map(l, 0, list(range(cfg.M)), host(b13), host(b2))
            del b13, b2
            for a in range(cfg.N):
                a13, a2 = wl.stacked_expert_weights(cfg, l, a + 1, len(tuned[a]))
                self.pool.map(l, a + 1, [int(e) for e in tuned[a]], host(a13) if len(tuned[a]) else None,
                              host(a2) if len(tuned[a]) else None)
            gates.append(dev(wl.gate_weight(cfg, l)))
            sh13, sh2 = wl.shared_weights(cfg, l)
            shared.append((dev(sh13), dev(sh2)))
            if l % 5 == 4:
                print(f"[bench]   layer {l + 1}/{L} loaded, {time.time() - t0:.0f} s", file=sys.stderr, flush=True)
        self.stack = layer_mod.MoEStack(self.pool, gates, shared, cfg.k, cfg.I, cfg.T, torch.bfloat16)
        self.x = dev(wl.tokens(cfg))
        self.aid = dev(wl.adapter_ids(cfg))
        self.aid0 = torch.zeros_like(self.aid)
        torch.cuda.synchronize()
        self.setup_s = time.time() - t0

    def active_slots(self, aid):
        """Sum over layers of the slots with at least one row (one untimed pass, layer by layer)."""
        h, total = self.x, 0
        for l in range(self.cfg.L):
            h = self.stack.forward(h, aid, first=l, last=l + 1)
            total += int((self.stack.layers[l].counts > 0).sum().item())
        return total

    def time_steps(self, steps, warmup, aid):
        return timed_steps(lambda: self.stack.forward(self.x, aid), steps, warmup)

    def time_graph_steps(self, steps, warmup, aid):
        """The same step captured once in a HIP graph and replayed (the step enqueues kernels only); checks the
        replayed result against the eager one bit for bit."""
        want = self.stack.forward(self.x, aid).clone()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            self.stack.forward(self.x, aid)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            out = self.stack.forward(self.x, aid)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        if not torch.equal(out, want):
            raise RuntimeError("graph replay differs from the eager step")
        return timed_steps(g.replay, steps, warmup)


def cpu_baseline(cfg):
    """The CPU oracle, as it stands, on the whole workload of the headline configuration (about 10-30 s on the GPU
    box's host cores, BLAS threads = the cores the process may use), plus the integer stages of the rerouting
    microbenchmark (configuration 3: lookup, counts, offsets, stable permutation) on one thread."""
    from oracle import moe
    tuned = wl.tuned_sets(cfg)
    x, aid, Wg = wl.tokens(cfg), wl.adapter_ids(cfg), wl.gate_weight(cfg)
    base = wl.stacked_expert_weights(cfg, 0, 0, cfg.M)
    adapters = [wl.stacked_expert_weights(cfg, 0, a + 1, len(tuned[a])) for a in range(cfg.N)]
    shared = wl.shared_weights(cfg)
    bias = wl.logit_bias_table(cfg, tuned) if cfg.gate_bias else None
    t0 = time.perf_counter()
    logits = moe.gate_logits(x, Wg, aid, bias)
    moe.moe_layer(x, logits, aid, cfg.k, cfg.M, cfg.N, cfg.E_max, tuned, base, adapters, shared)
    dt = time.perf_counter() - t0
    cores = len(os.sched_getaffinity(0))
    del base, adapters
    c3 = wl.get_config(3)
    ids3, aid3 = wl.distinct_topk_ids(c3), wl.adapter_ids(c3)
    emap3 = moe.build_expert_map(c3.M, c3.N, c3.E_max, wl.tuned_sets(c3))
    from threadpoolctl import threadpool_limits
    with threadpool_limits(limits=1):
        t0 = time.perf_counter()
        moe.permute(moe.reroute(ids3, aid3, emap3), c3.P)
        dt3 = time.perf_counter() - t0
    return {"value": cfg.T / dt, "unit": "tokens/s", "cores": cores, "kind": "oracle",
            "sample": f"all {cfg.T} tokens of {cfg.name}, one layer step (numpy fp64 oracle, {dt:.1f} s wall, BLAS threads = cores)",
            "integer_stages_c3": {"value": c3.T / dt3, "unit": "tokens/s", "cores": 1, "kind": "oracle",
                                  "sample": f"all {c3.T} tokens of {c3.name}: rerouting + counts + offsets + stable "
                                            f"permutation (numpy, {dt3:.2f} s wall, one thread)"}}


def table1_pool_stats(ew):
    """The paper's Table 1 adapters (max / average tuned experts per layer, L = 26, M = 64) as synthetic per-layer counts
    in a host-memory pool with N = 10, E_max = 13 (Sec. 3.1): F_mem and physical bytes, virtual tensor against padding."""
    rows = []
    with open(os.path.join(ROOT, "tests", "golden", "table1_adapter_sparsity.txt")) as f:
        for line in f:
            if line.strip() and not line.startswith("#"):
                name, mx, avg, _ = line.split()
                rows.append((name, int(mx), float(avg)))
    rng = np.random.default_rng(26)
    L, M, N, E_max, page, eb13, eb2 = 26, 64, len(rows), 13, 4096, 22528, 11264   # expert = 5.5 + 2.75 pages, as at 2 MiB
    out = {}
    pools = {m: ew.ExpertPool(L, M, N, E_max, eb13, eb2, page_bytes=page, flags=ew.EW_POOL_FAKE | f)
             for m, f in (("virtual_tensor", 0), ("padded", ew.EW_POOL_PADDED))}
    for i, (name, mx, avg) in enumerate(rows):
        e = np.full(L, mx, dtype=np.int64)
        while e.sum() > round(avg * L):
            l = int(rng.integers(1, L))
            e[l] -= e[l] > 0
        for l in range(L):
            for pool in pools.values():
                if i == 0:
                    pool.map(l, 0, list(range(M)))
                pool.map(l, i + 1, list(range(int(e[l]))))
    for m, pool in pools.items():
        st = pool.stats()
        out[m] = {"f_mem": st["f_mem"], "pages_mapped": st["pages_mapped"], "experts_loaded": st["experts_loaded"]}
        pool.close()
    out["physical_bytes_padded_over_virtual"] = out["padded"]["pages_mapped"] / out["virtual_tensor"]["pages_mapped"]
    out["paper_f_mem"] = 1.51
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extras", action="store_true", help="skip the decode (C1) and 26-layer stack (C4) legs")
    ap.add_argument("--no-stack", action="store_true", help="skip the 26-layer stack (C4) leg (about 110 GB of weights)")
    ap.add_argument("--ffn-only", choices=["c1", "c2"], default=None,
                    help="profiling aid: load that configuration, route once, then time only the routed moe_grouped_ffn "
                         "call --steps times (so rocprofv3's per-kernel averages cover exactly the launches of `roofline`)")
    ap.add_argument("--reroute-only", action="store_true",
                    help="profiling aid: only the fused rerouting + permutation of the integer microbenchmark (configuration 3)")
    ap.add_argument("--stack-only", action="store_true",
                    help="profiling aid: load the 26-layer stack (C4) and time only its decode step, 20 adapters then base-only")
    ap.add_argument("--peaks-only", action="store_true", help="run only the measured-peaks leg (stream read, copy, MFMA loops)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="run only five 1 GiB device-to-device tensor copies (a plain copy kernel of known size, for "
                         "scaling rocprofv3's FETCH_SIZE / WRITE_SIZE counters) and exit")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on one GPU only (no sharding or collectives); use --gpus 1", file=sys.stderr)
        sys.exit(2)
    if not torch.cuda.is_available():
        print("bench.py: no GPU visible; the HIP path has no CPU fallback", file=sys.stderr)
        sys.exit(1)

    if args.calibrate_copy:
        src = torch.full((1 << 28,), 1.0, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(5):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"calibrate_copy": {"bytes_read_per_copy": src.numel() * 4, "bytes_written_per_copy": src.numel() * 4,
                                             "copies": 5}}))
        return

    import paper_2508_17624_amd as ew
    from paper_2508_17624_amd import binding as B, layer as layer_mod
    lib_ = ew.lib()

    if args.peaks_only:
        print(json.dumps({"measured_peaks": measured_peaks(B, lib_)}))
        return

    if args.reroute_only:
        c3 = wl.get_config(3)
        T, k, P, N, E = c3.T, c3.k, c3.P, c3.N, c3.M
        i32 = dict(dtype=torch.int32, device="cuda")
        pool3, emap_ptr = c3_pool(c3)
        ids, aid = dev(wl.distinct_topk_ids(c3)), dev(wl.adapter_ids(c3))
        slot, counts, offsets = torch.empty((T, k), **i32), torch.empty(P, **i32), torch.empty(P + 1, **i32)
        por, rop = torch.empty(T * k, **i32), torch.empty(T * k, **i32)
        ws = B._workspace(lib_.moe_reroute_permute_workspace_bytes(T, k, P), "cuda")
        st = B._stream()
        t, tm = time_call(lambda: B._check(lib_.moe_reroute_permute(
            ids.data_ptr(), aid.data_ptr(), emap_ptr, T, k, E, N, P, slot.data_ptr(), counts.data_ptr(), offsets.data_ptr(),
            por.data_ptr(), rop.data_ptr(), ws.data_ptr(), ws.numel(), st)), iters=args.steps)
        alg = T * (4.0 * k + 4 + 3 * 4.0 * k)                 # ids + adapter id read; slots and both indices written
        print(json.dumps({"reroute_only": c3.name, "launches": args.steps + 3, "tokens": T, "median_us": t * 1e6, "avg_us": tm * 1e6,
                          "algorithmic_bytes": alg, "GB/s": alg / tm / 1e9}))
        return

    if args.stack_only:
        c4 = wl.get_config(4)
        s4 = StackSetup(c4, ew, layer_mod)
        a4, a4b = s4.active_slots(s4.aid), s4.active_slots(s4.aid0)
        t4, t4_med = s4.time_steps(args.steps, 3, s4.aid)
        t4b, t4b_med = s4.time_steps(args.steps, 3, s4.aid0)
        per = 3.0 * c4.H * c4.I * 2
        print(json.dumps({"stack_only": c4.name, "layers": c4.L, "steps": args.steps + 3, "active_slots_sum": a4,
                          "ms_per_step": t4 * 1e3, "median_ms_per_step": t4_med * 1e3,
                          "GB/s": (a4 + c4.S * c4.L) * per / t4 / 1e9,
                          "base_only": {"active_slots_sum": a4b, "ms_per_step": t4b * 1e3, "median_ms_per_step": t4b_med * 1e3,
                                        "GB/s": (a4b + c4.S * c4.L) * per / t4b / 1e9}}))
        return

    if args.ffn_only:
        cfg = wl.get_config(2 if args.ffn_only == "c2" else 1)
        s = LayerSetup(cfg, ew, layer_mod)
        s.layer.route(s.x, s.aid)
        torch.cuda.synchronize()
        active = s.active_slots()
        avg, med = s.time_ffn(args.steps, B)
        flops, wbytes = s.ffn_work(active)
        print(json.dumps({"ffn_only": cfg.name, "launches": args.steps + 3, "active_slots": active, "avg_ms": avg * 1e3,
                          "median_ms": med * 1e3, "TFLOP/s": flops / avg / 1e12, "GB/s": wbytes / avg / 1e9}))
        return

    cfg = wl.get_config(2)
    print(f"[bench] loading {cfg.name} ...", file=sys.stderr, flush=True)
    s2 = LayerSetup(cfg, ew, layer_mod)
    print(f"[bench] loaded in {s2.setup_s:.1f} s; pool {s2.pool.stats()}", file=sys.stderr, flush=True)

    t_step, t_step_med = s2.time_steps(args.steps, args.warmup)
    active = s2.active_slots()
    t_ffn_avg, t_ffn_med = s2.time_ffn(min(args.steps, 30), B)
    flops_ffn, wbytes2 = s2.ffn_work(active)
    t_base, t_base_med = s2.time_steps(args.steps, args.warmup, s2.aid0)
    active_base = s2.active_slots()
    t_ffn_base_avg, _ = s2.time_ffn(min(args.steps, 30), B)
    s2.step()  # leave 20-adapter state
    peaks = measured_peaks(B, lib_)
    byte_ratio2 = (active + cfg.S) / (active_base + cfg.S)
    mfma_meas = peaks["mfma_bf16_random_operands_TFLOPs"]

    result = {
        "metric": "MoE-layer tokens/s at 20 adapters (1 GPU)",
        "value": cfg.T / t_step,
        "unit": "tokens/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": t_step * 1e3,
        "median_ms_per_step": t_step_med * 1e3,         # median over the same steps of per-step HIP-event pairs
        "value_at_median": cfg.T / t_step_med,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16", "data": "synthetic",
        "config": {"workload": cfg.name, "tokens": cfg.T, "hidden": cfg.H, "experts": cfg.M, "intermediate": cfg.I,
                   "shared_experts": cfg.S, "top_k": cfg.k, "adapters": cfg.N, "E_max": cfg.E_max, "slots": cfg.P,
                   "active_slots": active, "pool": "vmm"},
        "roofline": {"bound": "mfma", "kernel": "moe_grouped_ffn_with_shared: routed + shared experts (k_ffn_plan, k_ffn_big: both products in one launch)",
                     "achieved": flops_ffn / t_ffn_avg / 1e12, "peak": MFMA_BF16_PEAK_TFLOPS, "unit": "TFLOP/s",
                     "frac": flops_ffn / t_ffn_avg / 1e12 / MFMA_BF16_PEAK_TFLOPS, "traffic": traffic_bytes(cfg.name),
                     "measured_peak": mfma_meas, "frac_of_measured": flops_ffn / t_ffn_avg / 1e12 / mfma_meas,
                     "hbm_view": {"algorithmic_weight_bytes": wbytes2, "achieved_GBs": wbytes2 / t_ffn_avg / 1e9,
                                  "peak_GBs": HBM_PEAK_GBS, "frac": wbytes2 / t_ffn_avg / 1e9 / HBM_PEAK_GBS,
                                  "measured_peak_GBs": peaks["hbm_read_GBs"],
                                  "frac_of_measured": wbytes2 / t_ffn_avg / 1e9 / peaks["hbm_read_GBs"]},
                     "avg_ms": t_ffn_avg * 1e3, "median_ms": t_ffn_med * 1e3,
                     "base_only_ffn": {"avg_ms": t_ffn_base_avg * 1e3, "TFLOPs": flops_ffn / t_ffn_base_avg / 1e12,
                                              "frac": flops_ffn / t_ffn_base_avg / 1e12 / MFMA_BF16_PEAK_TFLOPS}},
        "measured_peaks": peaks,
        "stage_us": s2.stage_us(B),
        "overhead_vs_base_only_pct": (t_step / t_base - 1.0) * 100.0,
        "overhead_per_byte_pct": ((t_step / t_base) / byte_ratio2 - 1.0) * 100.0,
        "base_only": {"ms_per_step": t_base * 1e3, "median_ms_per_step": t_base_med * 1e3, "active_slots": active_base,
                      "weight_bytes_ratio": byte_ratio2},
    }

    if not args.no_extras:
        c1 = wl.get_config(1)
        print(f"[bench] loading {c1.name} ...", file=sys.stderr, flush=True)
        s1 = LayerSetup(c1, ew, layer_mod)
        t1, t1_med = s1.time_steps(max(args.steps, 100), args.warmup)
        a1 = s1.active_slots()
        f_avg, f_med = s1.time_ffn(50, B)
        # cold figure: 1.44 GB of weights exceed the 256 MB memory-side cache, but a part of them can still hit it from
        # one call to the next; a 1 GiB streaming read between the calls evicts both cache levels
        fl_src = torch.empty(1 << 30, dtype=torch.uint8, device="cuda").zero_()
        fl_dst = torch.empty(256, dtype=torch.uint8, device="cuda")
        st_ = B._stream()
        f_cold = s1.time_ffn_cold(B, lambda: B._check(lib_.ew_probe_stream(fl_src.data_ptr(), fl_dst.data_ptr(), 1 << 30, 1, st_)))
        del fl_src
        stage1 = s1.stage_us(B, iters=50)
        t1b, t1b_med = s1.time_steps(max(args.steps, 100), args.warmup, s1.aid0)
        a1b = s1.active_slots()
        _, wbytes = s1.ffn_work(a1)
        ratio1 = (a1 + c1.S) / (a1b + c1.S)
        result["extras"] = {"decode_c1": {
            "workload": c1.name, "tokens_per_s": c1.T / t1, "ms_per_step": t1 * 1e3, "median_ms_per_step": t1_med * 1e3,
            "active_slots": a1, "stage_us": stage1,
            "roofline": {"bound": "hbm", "kernel": "moe_grouped_ffn_with_shared: routed + shared experts (k_ffn_plan, k_ffn_dec<4, ...>: both products in one launch)",
                         "achieved": wbytes / f_avg / 1e9,
                         "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": wbytes / f_avg / 1e9 / HBM_PEAK_GBS,
                         "measured_peak": peaks["hbm_read_GBs"], "frac_of_measured": wbytes / f_avg / 1e9 / peaks["hbm_read_GBs"],
                         "traffic": traffic_bytes(c1.name), "avg_ms": f_avg * 1e3, "median_ms": f_med * 1e3,
                         "cold_caches_median_ms": f_cold * 1e3, "cold_caches_GBs": wbytes / f_cold / 1e9,
                         "cold_caches_frac": wbytes / f_cold / 1e9 / HBM_PEAK_GBS},
            "overhead_vs_base_only_pct": (t1 / t1b - 1.0) * 100.0,
            "overhead_per_byte_pct": ((t1 / t1b) / ratio1 - 1.0) * 100.0,
            "base_only": {"ms_per_step": t1b * 1e3, "median_ms_per_step": t1b_med * 1e3, "active_slots": a1b,
                          "weight_bytes_ratio": ratio1,
                          "achieved_GBs": (a1b + c1.S) * 3.0 * c1.H * c1.I * 2 / t1b / 1e9}}}
        print("[bench] rerouting ablation, pool modes, adapter churn, second workload ...", file=sys.stderr, flush=True)
        try:
            result["extras"]["ablation_rerouting"] = ablation_rerouting(B, lib_, s2, t_step, s1, t1)
        except Exception as e:  # report, keep the headline
            result["extras"]["ablation_error"] = f"{type(e).__name__}: {e}"
        s1.pool.close()
        del s1
        try:
            result["extras"]["second_workload_sweep"] = second_workload_sweep(s2)
            result["extras"]["pool_modes_c1"] = pool_modes(B, lib_, ew, layer_mod, c1, 50)
            result["extras"]["adapter_churn_c1"] = {"lazy_unmap": adapter_churn(ew, c1, 0),
                                                    "eager_unmap": adapter_churn(ew, c1, ew.EW_POOL_EAGER_UNMAP)}
            result["extras"]["table1_adapters_pool_stats"] = table1_pool_stats(ew)
        except Exception as e:  # report, keep the headline
            result["extras"]["next_rows_error"] = f"{type(e).__name__}: {e}"
        if not args.no_stack:
            s2.pool.close()
            c4 = wl.get_config(4)
            print(f"[bench] loading {c4.name} ({c4.L} layers) ...", file=sys.stderr, flush=True)
            try:
                s4 = StackSetup(c4, ew, layer_mod)
                st4 = s4.pool.stats()
                a4, a4b = s4.active_slots(s4.aid), s4.active_slots(s4.aid0)
                n4 = max(5, min(args.steps, 20))
                t4, t4_med = s4.time_steps(n4, 3, s4.aid)
                t4b, t4b_med = s4.time_steps(n4, 3, s4.aid0)
                try:
                    t4g, _ = s4.time_graph_steps(n4, 3, s4.aid)
                except Exception as e:  # report, keep the eager figures
                    t4g = None
                    print(f"[bench] graph replay of the stack failed: {type(e).__name__}: {e}", file=sys.stderr, flush=True)
                per = 3.0 * c4.H * c4.I * 2
                wb, wbb = (a4 + c4.S * c4.L) * per, (a4b + c4.S * c4.L) * per
                result["extras"]["stack_c4"] = {
                    "workload": c4.name, "layers": c4.L, "tokens_per_s": c4.T / t4, "ms_per_step": t4 * 1e3,
                    "median_ms_per_step": t4_med * 1e3, "graph_replay_ms_per_step": t4g * 1e3 if t4g else None,
                    "active_slots_sum": a4, "setup_s": s4.setup_s,
                    "pool": {"page_bytes": st4["page_bytes"], "pages_mapped": st4["pages_mapped"],
                             "bytes_experts": st4["bytes_experts"], "bytes_virtual": st4["bytes_virtual"], "f_mem": st4["f_mem"]},
                    "roofline": {"bound": "hbm", "kernel": "whole decode step (weights of active slots + shared experts)",
                                 "achieved": wb / t4 / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": wb / t4 / 1e9 / HBM_PEAK_GBS,
                                 "measured_peak": peaks["hbm_read_GBs"], "frac_of_measured": wb / t4 / 1e9 / peaks["hbm_read_GBs"]},
                    "overhead_vs_base_only_pct": (t4 / t4b - 1.0) * 100.0,
                    "base_only": {"ms_per_step": t4b * 1e3, "median_ms_per_step": t4b_med * 1e3, "active_slots_sum": a4b,
                                  "weight_bytes_ratio": wb / wbb, "achieved_GBs": wbb / t4b / 1e9,
                                  "frac": wbb / t4b / 1e9 / HBM_PEAK_GBS},
                    "overhead_per_byte_pct": ((t4 / t4b) / (wb / wbb) - 1.0) * 100.0}
                s4.pool.close()
            except Exception as e:  # report, keep the headline
                result["extras"]["stack_c4"] = {"error": f"{type(e).__name__}: {e}"}

    if not args.no_cpu_baseline:
        print("[bench] timing the CPU oracle ...", file=sys.stderr, flush=True)
        result["cpu_baseline"] = cpu_baseline(cfg)
    else:
        result["cpu_baseline"] = None
    print(json.dumps(result))


if __name__ == "__main__":
    main()
