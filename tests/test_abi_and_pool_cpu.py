"""CPU-only checks of the C-ABI library: it loads, exports every declared symbol, validates
arguments on the host, and its expert pool (fake VMM backend: mmap + mprotect) keeps the page
accounting the oracle predicts, including failure injection and rollback."""
import ctypes as C
import os
import re

import numpy as np
import pytest
import torch

import paper_2508_17624_amd as ew
from oracle import moe, pool as opool

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = ew.EW_POOL_FAKE


def declared_functions():
    text = open(os.path.join(ROOT, "include", "expertweave.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return re.findall(r"\b([a-z_0-9]+)\s*\([^;{]*\)\s*;", text)


def test_library_exports_every_declared_symbol():
    lib = ew.lib()
    names = declared_functions()
    assert {"moe_route_topk", "moe_reroute_permute", "moe_grouped_ffn", "moe_unpermute", "expert_pool_map"} <= set(names)
    for n in names:
        assert hasattr(lib, n), f"{n} declared in expertweave.h but not exported"
        assert n in ew.binding.SIGNATURES, f"{n} has no binding signature"
    assert lib.ew_abi_version() == 4 and lib.ew_last_error() is not None


def test_host_side_argument_checks_need_no_gpu():
    lib = ew.lib()
    assert lib.moe_route_topk(None, 4, 8, 9, 0, None, None, None) == -1          # k > E
    assert b"k<=E" in lib.ew_last_error()
    assert lib.moe_route_topk(None, 4, 2048, 2, 0, None, None, None) == -6       # E above the limit
    assert lib.moe_route_topk(None, 0, 8, 2, 0, None, None, None) == 0           # empty batch: no-op
    assert lib.moe_reroute_permute(None, None, None, 4, 2, 8, 0, 4096, None, None, None, None, None, None, 0, None) == -6
    assert lib.moe_reroute_permute(None, None, None, 4, 2, 8, 0, 8, None, None, None, None, None, None, 0, None) == -1
    assert lib.moe_grouped_ffn(None, 7, 4, 2, 256, 128, 8, None, None, None, None, None, None, None, 0, None) == -1
    assert lib.moe_unpermute(None, None, None, None, 0, None, 4, 2, 100, ew.EW_BF16, None, None) == -6   # H % 8
    assert lib.moe_reroute_permute_workspace_bytes(64, 6, 128) == 4 * 128 * 4      # 4 blocks of 16 tokens x P counters
    assert lib.moe_reroute_permute_workspace_bytes(0, 6, 128) == 0                # empty batch
    assert lib.moe_reroute_singleop_workspace_bytes(64, 6) == 2 * 1536
    assert lib.moe_reroute_singleop(None, None, None, 4, 2, 8, 0, None, None, 0, None) == -1
    assert lib.moe_reroute_permute_workspace_bytes(1 << 20, 6, 384) > 0
    need = lib.moe_grouped_ffn_workspace_bytes(64, 6, 2048, 1408, 128, ew.EW_BF16)
    assert need >= 64 * 6 * 1408 * 2 and need % 256 == 0


@pytest.mark.parametrize("dtype", [ew.EW_F32, ew.EW_BF16])
@pytest.mark.parametrize("I", [1, 4, 128])
def test_ffn_workspace_never_shrinks_with_more_tokens(dtype, I):
    """A workspace made for the largest batch serves every smaller one, also where the work plan's chunk size changes."""
    size = ew.lib().moe_grouped_ffn_workspace_bytes
    for k in (1, 2, 6, 9, 16):
        for P in (1, 3, 7, 40, 386, 2048):
            need = [size(T, k, 128, I, P, dtype) for T in (*range(1, 140), 511, 512, 513, 4096, 65536)]
            assert all(a <= b for a, b in zip(need, need[1:])), (k, P)


def test_layer_forward_checks_its_arguments_before_any_launch():
    """Errors that need no GPU: what is refused here has enqueued nothing (a launch would fail differently, and with logits
    given no earlier step looks at the type)."""
    lib = ew.lib()
    one = C.c_void_p(256)                                       # never dereferenced

    def call(T=4, logits=one, **kw):
        d = dict(dtype=ew.EW_F32, H=64, I=32, M=8, k=2, N=1, P=16, S=1, T_max=1 << 30)
        d.update({n: 256 for n, t in ew.binding.LayerDesc._fields_ if t is C.c_void_p})
        d.update(ws_perm_bytes=1 << 40, ws_ffn_bytes=1 << 40, **kw)
        return lib.moe_layer_forward(C.byref(ew.binding.LayerDesc(**d)), one, one, T, logits, None, one, None, 0.0, None)

    assert lib.moe_layer_forward(None, one, one, 4, one, None, one, None, 0.0, None) == -1
    for dtype in (2, 7, -1):
        assert call(dtype=dtype) == -1 and b"dtype" in lib.ew_last_error()
        assert call(dtype=dtype, logits=None) == -1
    assert call(T=-1) == -1 and call(T=9, T_max=8) == -1
    for field in ("k", "H", "I", "P"):
        assert call(**{field: 0}) == -1
    assert call(S=-1) == -1
    # each row count of its own below 2^31, the sum not
    assert call(T=1 << 29, k=2, S=2) == -6 and b"2^31" in lib.ew_last_error()
    assert call(T=1 << 29, k=2, S=2, dtype=ew.EW_BF16, H=128, I=128) == -6


@pytest.mark.parametrize("H,I", [(32768, 32768), (1 << 20, 1024), (128, 1 << 23)])
def test_ffn_refuses_experts_beyond_its_weight_offsets(H, I):
    """The kernels keep a lane's offset into a slot's gate and up rows in 32 bits: 4*H*I bytes must stay below 2^32."""
    lib, one, T, k, P, S = ew.lib(), C.c_void_p(256), 1, 1, 2, 1
    big = 1 << 50
    for s in (0, S):
        args = (one, ew.EW_BF16, T, k, H, I, P, s, one, one, one, one, one, one, one, one, one, big, None)
        assert lib.moe_grouped_ffn_planned(*args) == -6 and b"2^30" in lib.ew_last_error()
        assert lib.moe_route_reroute_permute_plan(one, one, one, T, 8, k, 1, P, 0, one, one, one, one, one, one, one, one, big, H, I, s,
                                                  ew.EW_BF16, one, big, None) == -6
    assert lib.moe_grouped_ffn_with_shared(*args) == -6
    assert lib.moe_grouped_ffn(one, ew.EW_BF16, T, k, H, I, P, one, one, one, one, one, one, one, big, None) == -6


def test_pool_create_rejects_bad_arguments():
    for kw in (dict(num_layers=0), dict(M=0), dict(N=-1), dict(w13_bytes=0), dict(page_bytes=1000), dict(flags=64 | FAKE)):
        args = dict(num_layers=1, M=4, N=2, E_max=2, w13_bytes=4096, w2_bytes=4096, page_bytes=4096, flags=FAKE)
        args.update(kw)
        with pytest.raises(ew.EWError) as e:
            ew.ExpertPool(**args)
        assert e.value.code == -1


def _read(ptr, n):
    return np.frombuffer((C.c_uint8 * n).from_address(ptr), dtype=np.uint8).copy()


def test_fig3_example_through_the_pool(golden_fig3):
    """Paper Fig. 3: E_max=3, e_0=2, e_1=1, an expert is 1.5 pages -> 3 pages under adapter 0."""
    g = golden_fig3
    page, M = 4096, 4
    eb = g["expert_pages_times_2"] * page // 2
    p = ew.ExpertPool(1, M, 2, g["E_max"], eb, eb, page_bytes=page, flags=FAKE)
    p.map(0, 0, list(range(M)))
    s0 = p.stats()["pages_mapped"]
    p.map(0, 1, list(range(g["e_0"])))
    assert p.stats()["pages_mapped"] - s0 == 2 * g["pages_adapter_0"]            # two tensors (W13 and W2)
    p.map(0, 2, list(range(g["e_1"])))
    assert p.stats()["pages_mapped"] - s0 == 2 * (g["pages_adapter_0"] + 2)
    pad0 = (M + g["e_0"]) * eb                                                    # first padding slot of adapter 1
    assert not p.fake_is_mapped(0, 0, pad0) and p.fake_is_mapped(0, 0, pad0 - 1)
    assert p.fake_is_mapped(0, 0, (M + g["E_max"]) * eb)                          # adapter 2 starts mid-page
    p.close()


@pytest.mark.parametrize("eager", [False, True], ids=["lazy", "eager"])
@pytest.mark.parametrize("seed", range(4))
def test_pool_matches_oracle_under_random_load_evict(seed, eager):
    rng = np.random.default_rng(seed)
    page = 4096
    M, N, E_max = 6, 5, 4
    eb13, eb2 = int(rng.integers(3, 40)) * 512, int(rng.integers(3, 40)) * 512
    p = ew.ExpertPool(2, M, N, E_max, eb13, eb2, page_bytes=page, prealloc_pages=3,
                      flags=FAKE | (ew.EW_POOL_EAGER_UNMAP if eager else 0))
    ora = [[opool.VirtualTensorPages(p.P, eb, page) for eb in (eb13, eb2)] for _ in range(2)]
    loaded, tuned = {}, {}
    data = {}
    assert p.stats()["pages_free"] == 3
    for step in range(60):
        layer, a = int(rng.integers(2)), int(rng.integers(0, N + 1))
        if (layer, a) in loaded:
            p.unmap(layer, a)
            for vt in ora[layer]:
                vt.unload(0 if a == 0 else M + (a - 1) * E_max)
            del loaded[(layer, a)]; tuned.pop((layer, a), None)
        else:
            n = M if a == 0 else int(rng.integers(0, E_max + 1))
            ids = list(range(M)) if a == 0 else sorted(rng.choice(M, n, replace=False).tolist())
            w13 = torch.from_numpy(rng.integers(0, 255, n * eb13, dtype=np.uint8))
            w2 = torch.from_numpy(rng.integers(0, 255, n * eb2, dtype=np.uint8))
            p.map(layer, a, ids, w13 if n else None, w2 if n else None)
            for vt in ora[layer]:
                vt.load(0 if a == 0 else M + (a - 1) * E_max, n)
            loaded[(layer, a)] = n
            data[(layer, a)] = (w13.numpy(), w2.numpy())
            if a:
                tuned[(layer, a)] = ids
        st = p.stats()
        want_pages = sum(len(vt.mapped_pages()) for l in ora for vt in l)
        assert st["pages_mapped"] == want_pages
        assert st["pages_shared"] == sum(len(vt.shared_pages()) for l in ora for vt in l)
        assert st["pages_created"] - st["pages_released"] == st["pages_mapped"] + st["pages_free"] + st["pages_parked"]
        assert not eager or st["pages_parked"] == 0
        assert st["experts_loaded"] == sum(loaded.values())
        # every loaded range still holds exactly the bytes that were copied in; maps match the oracle
        for layer in range(2):
            w13b, w2b, emap_ptr, P = p.view(layer)
            for (l, a), n in loaded.items():
                if l != layer or n == 0:
                    continue
                s0 = 0 if a == 0 else M + (a - 1) * E_max
                np.testing.assert_array_equal(_read(w13b + s0 * eb13, n * eb13), data[(l, a)][0])
                np.testing.assert_array_equal(_read(w2b + s0 * eb2, n * eb2), data[(l, a)][1])
            t = [tuned.get((layer, a), []) for a in range(1, N + 1)]
            np.testing.assert_array_equal(p.expert_map_host(layer).numpy(), moe.build_expert_map(M, N, E_max, t))
            np.testing.assert_array_equal(np.frombuffer((C.c_int32 * ((N + 1) * M)).from_address(emap_ptr), dtype=np.int32)
                                          .reshape(N + 1, M), p.expert_map_host(layer).numpy())
            for which, vt in enumerate(ora[layer]):
                for q in range(vt.P * vt.expert_bytes // page):
                    assert p.fake_is_mapped(layer, which, q * page) == (q in vt.refs)
    for (layer, a) in list(loaded):
        p.unmap(layer, a)
    st = p.stats()
    assert st["pages_mapped"] == 0 and st["experts_loaded"] == 0 and st["f_mem"] == 0
    p.trim(0)
    st = p.stats()
    assert st["pages_free"] == 0 and st["pages_parked"] == 0 and st["pages_released"] == st["pages_created"]
    p.close()


def test_lazy_eviction_parks_pages_and_reuses_them():
    """Evicted pages stay mapped in place (parked): re-loading the same range needs no page at all, loading
    elsewhere takes the free list first and then moves the oldest parked page, trim unmaps them all."""
    page, M, N, E_max, eb = 4096, 4, 3, 2, 2 * 4096                  # an expert = 2 pages, slots page-aligned
    p = ew.ExpertPool(1, M, N, E_max, eb, eb, page_bytes=page, flags=FAKE)
    p.map(0, 0, list(range(M)))
    base = p.stats()
    assert base["pages_mapped"] == 2 * M * 2 and base["pages_parked"] == 0
    p.map(0, 1, [0, 1])                                               # 2 experts x 2 pages x 2 tensors = 8 pages
    created = p.stats()["pages_created"]
    p.unmap(0, 1)
    st = p.stats()
    assert st["pages_mapped"] == base["pages_mapped"] and st["pages_parked"] == 8 and st["pages_free"] == 0
    assert not p.fake_is_mapped(0, 0, M * eb)                         # logically gone at once
    assert p.expert_map_host(0)[1].tolist() == list(range(M))         # and unreachable: the row is identity again
    p.map(0, 1, [2])                                                  # same place, one expert: 4 parked pages come back
    st = p.stats()
    assert st["pages_created"] == created and st["pages_parked"] == 4 and st["pages_mapped"] == base["pages_mapped"] + 4
    p.map(0, 2, [0, 3])                                               # elsewhere: the 4 parked pages move, 4 are created
    st = p.stats()
    assert st["pages_parked"] == 0 and st["pages_created"] == created + 4 and st["pages_free"] == 0
    assert st["pages_created"] - st["pages_released"] == st["pages_mapped"]
    p.unmap(0, 2); p.unmap(0, 1)
    assert p.stats()["pages_parked"] == 12
    p.trim(2)
    st = p.stats()
    assert st["pages_parked"] == 0 and st["pages_free"] == 2 and st["pages_released"] == 10
    p.close()
    # churn of one adapter does not grow the parked queue without bound (stale entries are dropped)
    p = ew.ExpertPool(1, M, N, E_max, eb, eb, page_bytes=page, flags=FAKE)
    p.map(0, 0, list(range(M)))
    for _ in range(300):
        p.map(0, 1, [1, 2]); p.unmap(0, 1)
    st = p.stats()
    assert st["pages_parked"] == 8 and st["pages_created"] == base["pages_mapped"] + 8
    p.close()


@pytest.mark.parametrize("eager", [False, True], ids=["lazy", "eager"])
def test_failed_unmap_leaves_a_consistent_pool(eager):
    """A backend unmap that fails leaves the page mapped: the pool keeps its handle attached (parked) instead of
    recycling it, the page table and the statistics stay true, and later loads work."""
    page, M, N, E_max, eb = 4096, 4, 2, 2, 6144
    p = ew.ExpertPool(1, M, N, E_max, eb, eb, page_bytes=page, flags=FAKE | (ew.EW_POOL_EAGER_UNMAP if eager else 0))
    p.map(0, 0, list(range(M)))
    p.map(0, 1, [0, 1]); p.map(0, 2, [2])
    inv = lambda st: st["pages_created"] - st["pages_released"] == st["pages_mapped"] + st["pages_free"] + st["pages_parked"]
    if eager:
        p.fake_fail_at(2, 2)                                          # the second unmap of the eviction fails
        with pytest.raises(ew.EWError) as e:
            p.unmap(0, 1)
        assert e.value.code == -3
        st = p.stats()
        assert st["pages_parked"] == 1 and inv(st)                    # that page is still mapped, hence parked
    else:
        p.unmap(0, 1)
        p.fake_fail_at(2, 1)                                          # the first unmap of the trim fails
        with pytest.raises(ew.EWError) as e:
            p.trim(0)
        assert e.value.code == -3
        st = p.stats()
        assert st["pages_parked"] == 1 and st["pages_free"] == 0 and inv(st)
    assert p.expert_map_host(0)[1].tolist() == list(range(M))         # the adapter is evicted all the same
    with pytest.raises(ew.EWError) as e:
        p.unmap(0, 1)
    assert e.value.code == -4
    for off in range(M * eb, (M + E_max) * eb, page):                 # pages of the evicted range that nobody shares
        if off // page * page >= M * eb and off // page * page + page <= (M + E_max) * eb:
            assert not p.fake_is_mapped(0, 0, off)
    p.map(0, 1, [1, 3])                                               # takes the parked page back in place
    st = p.stats()
    assert st["pages_parked"] == 0 and inv(st)
    w13b, _, _, _ = p.view(0)
    C.memset(w13b + M * eb, 7, 2 * eb)                                # the whole range is writable memory
    p.unmap(0, 1); p.unmap(0, 2); p.unmap(0, 0)
    p.trim(0)
    st = p.stats()
    assert st["pages_mapped"] == 0 and st["pages_parked"] == 0 and st["pages_released"] == st["pages_created"]
    p.close()


def test_table1_shaped_adapters_through_the_pool(golden_table1):
    """The ten adapters of the paper's Table 1 (max and average tuned experts per layer, L = 26) as synthetic
    per-layer counts loaded into a pool with M = 64, N = 10, E_max = 13 (Sec. 3.1): the pool's F_mem reproduces
    the printed 1.51 to +-0.01 and equals the closed form on the same counts; the virtual tensor backs 29-40 %
    less adapter memory than padding every adapter to its own maximum (the saving Sec. 5.4 reports per adapter)."""
    rng = np.random.default_rng(26)
    L, M, N, E_max = 26, 64, 10, 13
    page, eb13, eb2 = 4096, 3 * 4096, 6144                            # 3 and 1.5 pages per expert: shared boundary pages
    counts = []                                                       # counts[i][l]
    for name, mx, avg, s in golden_table1:
        total = int(round(avg * L))
        assert abs(total - avg * L) < 0.14                            # the table prints the average to two decimals
        e = np.full(L, mx, dtype=np.int64)                            # start at the maximum, remove until the sum fits
        while e.sum() > total:
            l = int(rng.integers(1, L))                               # layer 0 stays at the maximum
            if e[l] > 0:
                e[l] -= 1
        assert e.max() == mx and e.sum() == total
        assert float(opool.adapter_sparsity(e)) == pytest.approx(s, abs=0.006)
        counts.append(e)
    p = ew.ExpertPool(L, M, N, E_max, eb13, eb2, page_bytes=page, flags=FAKE)
    pad = ew.ExpertPool(L, M, N, E_max, eb13, eb2, page_bytes=page, flags=FAKE | ew.EW_POOL_PADDED)
    for l in range(L):
        p.map(l, 0, list(range(M))); pad.map(l, 0, list(range(M)))
        for i in range(N):
            ids = sorted(rng.choice(M, int(counts[i][l]), replace=False).tolist())
            p.map(l, i + 1, ids); pad.map(l, i + 1, ids)
    st, stp = p.stats(), pad.stats()
    f_closed = float(opool.fragmentation_factor(M, N, E_max, [[int(counts[i][l]) for i in range(N)] for l in range(L)]))
    assert st["f_mem"] == pytest.approx(f_closed, rel=1e-12) and stp["f_mem"] == pytest.approx(f_closed, rel=1e-12)
    assert abs(st["f_mem"] - 1.51) <= 0.01                            # Sec. 3.1 prints 1.51
    assert st["experts_loaded"] == L * M + sum(int(c.sum()) for c in counts)
    # bytes: the virtual tensor maps the page cover of what is loaded, the padded pool everything
    per_expert = eb13 + eb2
    assert stp["pages_mapped"] * page >= L * (M + N * E_max) * per_expert
    ratio = (stp["pages_mapped"] * page) / (st["pages_mapped"] * page)
    assert ratio == pytest.approx(f_closed, rel=0.02)                 # physical bytes follow F_mem up to page rounding
    p.close(); pad.close()
    # Sec. 5.4: adapter memory under padding vs the virtual tensor for gate-math alone and for gate-math + token-math +
    # gate-intent (E_max = their largest per-layer count, 12).  Expert = 5.5 + 2.75 pages, the DeepSeek-V2-Lite expert
    # at 2 MiB pages.  The paper prints 40.4 % and 37.3 %; its two-adapter figure (28.9 %) follows from Table 1 for no
    # pair of these three (the closest, gate-math + gate-intent, gives 30.4 % here) and is not asserted.
    by_name = {row[0]: c for row, c in zip(golden_table1, counts)}
    eb13, eb2 = 22528, 11264
    for names, printed in ((["gate-math"], 0.404), (["gate-math", "token-math", "gate-intent"], 0.373)):
        E_max = max(int(by_name[n].max()) for n in names)
        mapped = {}
        for flags in (FAKE, FAKE | ew.EW_POOL_PADDED):
            q = ew.ExpertPool(L, M, len(names), E_max, eb13, eb2, page_bytes=page, flags=flags)
            for l in range(L):
                q.map(l, 0, list(range(M)))
            if flags == FAKE:
                base_pages = q.stats()["pages_mapped"]                 # what the base model alone needs
            for l in range(L):
                for i, n in enumerate(names):
                    q.map(l, i + 1, list(range(int(by_name[n][l]))))
            mapped[flags] = q.stats()["pages_mapped"]
            q.close()
        saving = 1.0 - (mapped[FAKE] - base_pages) / (mapped[FAKE | ew.EW_POOL_PADDED] - base_pages)
        assert saving == pytest.approx(printed, abs=0.02), (names, saving)


def test_pool_state_errors_and_rollback_on_injected_failures():
    page, M, N, E_max, eb = 4096, 4, 2, 3, 6144
    p = ew.ExpertPool(1, M, N, E_max, eb, eb, page_bytes=page, flags=FAKE)
    p.map(0, 0, list(range(M)))
    with pytest.raises(ew.EWError) as e:
        p.map(0, 0, list(range(M)))
    assert e.value.code == -4                                                     # double load
    with pytest.raises(ew.EWError) as e:
        p.unmap(0, 1)
    assert e.value.code == -4                                                     # evict of not-loaded
    for bad in ([1, 1], [2, 1], [4], [0, 1, 2, 3]):
        with pytest.raises(ew.EWError) as e:
            p.map(0, 1, bad)
        assert e.value.code == -1
    with pytest.raises(ew.EWError):
        p.map(0, 3, [0])                                                          # adapter id out of range
    with pytest.raises(ew.EWError):
        p.map(1, 1, [0])                                                          # layer out of range
    before = p.stats()
    map_before = p.expert_map_host(0).clone()
    for op, nth in ((0, 1), (0, 3), (1, 2), (1, 5)):                              # create / map fail at various points
        p.fake_fail_at(op, nth)
        with pytest.raises(ew.EWError) as e:
            p.map(0, 1, [0, 2, 3])
        assert e.value.code in (-2, -3) and "rolled back" in str(e.value)
        after = p.stats()
        assert after["pages_mapped"] == before["pages_mapped"] and after["experts_loaded"] == before["experts_loaded"]
        assert torch.equal(p.expert_map_host(0), map_before)
        for off in range(M * eb, (M + E_max) * eb, page):
            if off // page * page >= M * eb:                                      # pages not shared with the base range
                assert not p.fake_is_mapped(0, 0, off + page - 1 if off % page else off)
    p.fake_fail_at(0, 0)
    p.map(0, 1, [0, 2, 3])                                                        # and it works afterwards
    assert p.expert_map_host(0)[1].tolist() == [4, 1, 5, 6]
    p.close()


def test_padded_pool_backs_everything_and_f_mem():
    page, M, N, E_max, eb = 4096, 8, 2, 3, 4096
    p = ew.ExpertPool(3, M, N, E_max, eb, 2 * eb, page_bytes=page, flags=FAKE | ew.EW_POOL_PADDED)
    st = p.stats()
    assert st["pages_mapped"] == 3 * (p.P * 1 + p.P * 2)
    for l in range(3):
        p.map(l, 0, list(range(M)))
        p.map(l, 1, [1, 2, 3]); p.map(l, 2, [])
    st2 = p.stats()
    assert st2["pages_mapped"] == st["pages_mapped"] and st2["pages_shared"] == 0
    assert st2["f_mem"] == pytest.approx(float(opool.fragmentation_factor(M, N, E_max, [[3, 0]] * 3)))
    p.close()
    v = ew.ExpertPool(3, M, N, E_max, eb, 2 * eb, page_bytes=page, flags=FAKE)
    for l in range(3):
        v.map(l, 0, list(range(M))); v.map(l, 1, [1, 2, 3]); v.map(l, 2, [])
    assert v.stats()["pages_mapped"] == 3 * (M + 3) * 3                           # only loaded experts are backed
    v.close()


def test_lru_eviction_order_keeps_a_fixed_number_of_adapters_resident():
    """Adapter churn as a serving loop would drive it (paper Sec. 4.2): at most `cap` adapters resident, a batch
    touches its adapters, a missing adapter evicts the least recently used one.  The pool's victim choice is
    compared with a plain ordered-list LRU; after the run every page is accounted for."""
    rng = np.random.default_rng(11)
    M, N, E_max, cap, page = 6, 8, 3, 3, 4096
    p = ew.ExpertPool(2, M, N, E_max, 5 * 512, 3 * 512, page_bytes=page, flags=FAKE)
    for layer in range(2):
        p.map(layer, 0, list(range(M)))
    base_pages = p.stats()["pages_mapped"]
    assert p.lru_victim() == -1                                   # the base model is never a victim
    order = []                                                    # resident adapters, least recently used first
    for step in range(200):
        batch = sorted(set(int(a) for a in rng.integers(1, N + 1, size=int(rng.integers(1, 3)))))
        for a in batch:
            if a not in order:
                if len(order) == cap:
                    evictable = [v for v in order if v not in batch]   # order is LRU-first
                    victim = p.lru_victim()
                    if victim in batch:                             # the engine re-touches in-batch adapters first
                        p.touch([v for v in batch if v in order])
                        order = evictable + [v for v in order if v in batch]
                        victim = p.lru_victim()
                    assert victim == order[0]
                    for layer in range(2):
                        p.unmap(layer, victim)
                    order.remove(victim)
                n = int(rng.integers(0, E_max + 1))
                ids = sorted(rng.choice(M, n, replace=False).tolist())
                for layer in range(2):
                    p.map(layer, a, ids)
                order.append(a)
        p.touch([0] + batch)
        order = [v for v in order if v not in batch] + [v for v in batch]
        assert len(order) <= cap
    while order:
        v = p.lru_victim()
        assert v == order[0]
        for layer in range(2):
            p.unmap(layer, v)
        order.pop(0)
    assert p.lru_victim() == -1 and p.stats()["pages_mapped"] == base_pages
    with pytest.raises(ew.EWError):
        p.touch([N + 1])
    p.close()


def test_layer_description_follows_its_tensors():
    """A layer's description for moe_layer_forward names the storage that its weights and buffers have at the call, also
    when the storage changed under the same tensor object or a buffer was replaced."""
    from paper_2508_17624_amd.layer import MoELayer
    M, H, I, k, S, T = 4, 64, 32, 2, 1, 8
    p = ew.ExpertPool(1, M, 1, 2, 2 * I * H * 4, H * I * 4, flags=FAKE)
    sw13, sw2 = torch.zeros(S, 2 * I, H), torch.zeros(S, H, I)
    layer = MoELayer(p, 0, torch.zeros(M, H), sw13, sw2, k, I, T, torch.float32, bias=torch.zeros(2, M))

    def described():
        d = ew.binding.LayerDesc.from_address(layer._current())
        return d.Wg, d.bias, d.w13_shared, d.w2_shared, d.y, d.logits

    def actual():
        return tuple(t.data_ptr() for t in (layer.Wg, layer.bias, layer.shared_w13, layer.shared_w2, layer.buf.y, layer.buf.logits))

    assert described() == actual()
    layer.Wg.data, layer.bias.data = torch.ones(M, H), torch.ones(2, M)
    sw13.set_(torch.ones(S, 2 * I, H))
    sw2.data = torch.ones(S, H, I)
    assert described() == actual()
    layer.buf.y, layer.buf.logits = torch.zeros_like(layer.buf.y), torch.zeros_like(layer.buf.logits)
    layer.shared_w2 = torch.zeros(S, H, I)
    assert described() == actual()
    p.close()
