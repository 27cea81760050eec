"""GPU parity: router top-k, batched rerouting, permutation -- bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import moe

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ew():
    import paper_2508_17624_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.lib()
    return m


def _expert_map(cfg, layer=0):
    tuned = wl.tuned_sets(cfg, layer)
    return tuned, moe.build_expert_map(cfg.M, cfg.N, cfg.E_max, tuned)


def _check_permutation(got, ref_slot, P):
    slot, counts, offsets, por, rop = (t.cpu().numpy() for t in got)
    rc, ro, rp, rr = moe.permute(ref_slot, P)
    np.testing.assert_array_equal(slot, ref_slot)
    np.testing.assert_array_equal(counts, rc)
    np.testing.assert_array_equal(offsets, ro)
    np.testing.assert_array_equal(por, rp)
    np.testing.assert_array_equal(rop, rr)


@pytest.mark.parametrize("T,E,k", [(64, 8, 2), (64, 64, 6), (1000, 64, 6), (33, 160, 8), (7, 1024, 64), (1, 5, 5)])
@pytest.mark.parametrize("renorm", [False, True])
def test_route_topk(ew, T, E, k, renorm):
    rng = np.random.default_rng(T * 7 + E)
    logits = (rng.standard_normal((T, E)) * 1.5).astype(np.float32)
    ids, w = ew.moe_route_topk(torch.from_numpy(logits).cuda(), k, renorm)
    rids, rw = moe.route_topk(logits, k, renorm)
    np.testing.assert_array_equal(ids.cpu().numpy(), rids)
    np.testing.assert_allclose(w.cpu().numpy(), rw, rtol=2e-5, atol=1e-9)


def test_route_topk_ties_and_signed_zero(ew):
    rng = np.random.default_rng(5)
    logits = rng.integers(-2, 3, size=(512, 64)).astype(np.float32)       # many exact ties
    z = logits == 0
    logits[z] = np.where(rng.random(z.sum()) < 0.5, 0.0, -0.0)
    logits[0, :] = 1.25                                                    # all equal -> 0..k-1
    ids, w = ew.moe_route_topk(torch.from_numpy(logits).cuda(), 6)
    rids, rw = moe.route_topk(logits, 6)
    np.testing.assert_array_equal(ids.cpu().numpy(), rids)
    assert ids[0].tolist() == [0, 1, 2, 3, 4, 5]
    np.testing.assert_allclose(w.cpu().numpy(), rw, rtol=2e-5)


@pytest.mark.parametrize("E,k", [(1, 1), (16, 16), (17, 3), (64, 16), (64, 17), (65, 6), (128, 8), (129, 4), (256, 16), (257, 2)])
@pytest.mark.parametrize("T", [1, 4, 6, 67])
def test_route_topk_selection_edges(ew, T, E, k):
    """Both sides of every rule that picks a selection (experts per lane, choices per token) and tokens that do not fill a wave:
    ids exact with ties, both zeros, minus infinity and the largest values; the fused call gives the same bits."""
    rng = np.random.default_rng(1000 * E + k + T)
    logits = (rng.integers(-3, 4, size=(T, E)) * 0.5).astype(np.float32)
    logits[rng.random((T, E)) < 0.2] = -0.0
    logits[rng.random((T, E)) < 0.2] = -np.inf
    logits[:, rng.integers(E)] = np.float32(3e38) if T == 4 else np.float32(2.0)
    d = lambda a: torch.from_numpy(a).cuda()
    for renorm in (False, True):
        ids, w = ew.moe_route_topk(d(logits), k, renorm)
        rids, rw = moe.route_topk(logits, k, renorm)
        np.testing.assert_array_equal(ids.cpu().numpy(), rids)
        np.testing.assert_allclose(w.cpu().numpy(), rw, rtol=2e-5, atol=1e-9)
        emap = rng.permutation(E).astype(np.int32)[None]
        fused = ew.moe_route_reroute_permute(d(logits), torch.zeros(T, dtype=torch.int32, device="cuda"), d(emap), k, 0, E, renorm)
        assert torch.equal(fused[0], ids) and torch.equal(fused[1], w)
        _check_permutation(fused[2:], emap[0][rids], E)


@pytest.mark.parametrize("T,E,k", [(501, 1, 1), (501, 8, 2), (501, 16, 16), (501, 17, 3), (501, 48, 8), (501, 64, 6), (501, 65, 16), (501, 96, 4),
                                   (501, 128, 16), (501, 200, 5), (501, 256, 14), (1025, 129, 15), (1025, 256, 16)])
def test_route_topk_weights_do_not_depend_on_the_selection(ew, T, E, k):
    """Sixteen lanes per token and one wave per token give a weight the same bits: behind the E experts others that weigh exactly
    zero, up to the first number of experts that takes the wave; and the first tokens alone, where fewer of them take the wave."""
    rng = np.random.default_rng(E + k)
    logits = torch.from_numpy((rng.standard_normal((T, E)) * 1.5).astype(np.float32)).cuda()
    padded = torch.full((T, 257), -1e30, device="cuda")
    padded[:, :E] = logits
    for renorm in (False, True):
        ids, w = ew.moe_route_topk(logits, k, renorm)
        ids_w, w_w = ew.moe_route_topk(padded, k, renorm)
        assert torch.equal(ids, ids_w)
        assert torch.equal(w, w_w), f"{int((w != w_w).sum())} of {w.numel()} weights differ, renorm {renorm}"
        ids_f, w_f = ew.moe_route_topk(logits[:T - 1].contiguous(), k, renorm)
        assert torch.equal(ids[:T - 1], ids_f) and torch.equal(w[:T - 1], w_f)


@pytest.mark.parametrize("T,E,k", [((1 << 24) + 5, 2, 2), ((1 << 28) + 37, 1, 1), ((1 << 26) + 3, 17, 17)], ids=["second-stride", "sixteen-lanes", "wave"])
def test_route_topk_more_tokens_than_one_launch_has_threads_for(ew, T, E, k):
    """A few tokens more than fit a launch of less than 2^32 threads at sixteen lanes and at a wave per token, and more than the grid
    holds at once.  Logits 0 .. E-1 in an order that turns with the token: every choice of every token is known."""
    if torch.cuda.mem_get_info()[0] < 24 << 30:
        pytest.skip("needs 24 GB")
    B, step = ew.binding, 1 << 22
    e = torch.arange(E, device="cuda", dtype=torch.int32)
    turn = lambda t0: torch.arange(t0, min(T, t0 + step), device="cuda", dtype=torch.int32)[:, None] % E
    logits = torch.empty((T, E), device="cuda")
    for t0 in range(0, T, step):
        logits[t0:t0 + step] = ((e + turn(t0)) % E).float()
    ids, w = torch.full((T, k), -1, dtype=torch.int32, device="cuda"), torch.full((T, k), -1.0, device="cuda")
    B._check(B.lib().moe_route_topk(logits.data_ptr(), T, E, k, 0, ids.data_ptr(), w.data_ptr(), B._stream()))
    want_w = torch.softmax(torch.arange(E, dtype=torch.float64), 0).flip(0)[:k].float().cuda()
    for t0 in range(0, T, step):
        assert torch.equal(ids[t0:t0 + step], (E - 1 - e[:k] - turn(t0)) % E), f"ids from token {t0}"
        torch.testing.assert_close(w[t0:t0 + step], want_w.expand(min(step, T - t0), k), rtol=2e-5, atol=1e-9)


@pytest.mark.parametrize("T", [1, 64, 256, 341, 342, 682, 683, 1366, 2048, 2049, 5000])
def test_reroute_permute_configs(ew, T):
    """C2/C3-shaped: k=6, E=64, N=20, P=384.  T=341 is the last size of the single-block permutation
    (2048 pairs at most), 342 the first multi-block one; 2048 tokens fill one block's 12288 pairs
    exactly and 2049 spill into a second; 5000 spans several blocks with a ragged tail."""
    cfg = wl.get_config(3)
    tuned, emap = _expert_map(cfg)
    ids = wl.distinct_topk_ids(cfg, T)
    aid = wl.adapter_ids(cfg, T)
    got = ew.moe_reroute_permute(torch.from_numpy(ids).cuda(), torch.from_numpy(aid).cuda(),
                                 torch.from_numpy(emap).cuda(), cfg.N, cfg.P)
    _check_permutation(got, moe.reroute(ids, aid, emap), cfg.P)
    base = aid == 0
    assert np.array_equal(got[0].cpu().numpy()[base], ids[base])            # base tokens unchanged


@pytest.mark.parametrize("T,k,E,N,P", [(300, 1, 4, 0, 4), (100, 64, 64, 1, 128), (4000, 3, 2048, 0, 2048),
                                       (50, 2, 8, 2, 12), (9000, 5, 16, 3, 1)])
def test_reroute_permute_shapes_with_duplicates(ew, T, k, E, N, P):
    """Arbitrary expert maps (duplicate slots inside a token allowed): the sort stays stable."""
    rng = np.random.default_rng(T + k + P)
    ids = rng.integers(0, E, size=(T, k)).astype(np.int32)
    aid = rng.integers(0, N + 1, size=T).astype(np.int32)
    emap = rng.integers(0, P, size=(N + 1, E)).astype(np.int32)
    got = ew.moe_reroute_permute(torch.from_numpy(ids).cuda(), torch.from_numpy(aid).cuda(),
                                 torch.from_numpy(emap).cuda(), N, P)
    _check_permutation(got, moe.reroute(ids, aid, emap), P)


@pytest.mark.parametrize("T,E,k,P", [(32, 256, 16, 320), (33, 256, 16, 320), (33, 256, 15, 320), (128, 256, 16, 320), (129, 256, 16, 320),
                                     (33, 256, 4, 320), (33, 128, 12, 200), (48, 128, 12, 200), (48, 128, 13, 200), (49, 128, 4, 200), (49, 128, 5, 200),
                                     (64, 64, 8, 384), (64, 64, 9, 384), (65, 64, 6, 384), (28, 64, 8, 1600), (29, 64, 8, 1600), (29, 64, 9, 1600),
                                     (64, 16, 8, 2048), (64, 16, 9, 2048), (48, 64, 8, 2048), (49, 64, 8, 2048)])
def test_route_reroute_permute_joined_or_not(ew, T, E, k, P):
    """Both sides of every line between the selection inside the single block, in one to three rounds of its waves, and in a launch of
    its own."""
    rng = np.random.default_rng(T + E + k + P)
    logits = rng.standard_normal((T, E)).astype(np.float32)
    aid = rng.integers(0, 3, size=T).astype(np.int32)
    emap = np.stack([rng.choice(P, E, replace=False) for _ in range(3)]).astype(np.int32)
    d = lambda a: torch.from_numpy(a).cuda()
    got = ew.moe_route_reroute_permute(d(logits), d(aid), d(emap), k, 2, P)
    rids, rw = moe.route_topk(logits, k, False)
    np.testing.assert_array_equal(got[0].cpu().numpy(), rids)
    np.testing.assert_allclose(got[1].cpu().numpy(), rw, rtol=2e-5, atol=1e-9)
    _check_permutation(got[2:], moe.reroute(rids, aid, emap), P)


@pytest.mark.parametrize("T,k,E,P", [(600, 4, 32, 100), (2100, 2, 16, 128), (2100, 2, 16, 129), (5000, 3, 64, 256), (700, 7, 64, 257), (900, 5, 64, 512),
                                     (900, 5, 64, 513), (32768, 8, 64, 200), (32769, 8, 64, 200), (131072, 2, 16, 40), (131073, 2, 16, 40)])
def test_reroute_permute_two_or_three_launches(ew, T, k, E, P):
    """Both sides of the rules that choose them (2^18 pairs, 512 slots) and every width of the column sums; ids distinct inside a
    token as a top-k gives them, and a workspace sized for more tokens serves."""
    rng = np.random.default_rng(T + k + P)
    ids = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)
    aid = rng.integers(0, 3, size=T).astype(np.int32)
    emap = np.stack([rng.choice(P, E, replace=P < E) for _ in range(3)]).astype(np.int32)
    d = lambda a: torch.from_numpy(a).cuda()
    need = [ew.lib().moe_reroute_permute_workspace_bytes(t, k, P) for t in (T, T + 1, T + 17, 2 * T)]
    assert need == sorted(need)
    ws = torch.empty(need[1], dtype=torch.uint8, device="cuda")
    got = ew.moe_reroute_permute(d(ids), d(aid), d(emap), 2, P, ws=ws)
    _check_permutation(got, moe.reroute(ids, aid, emap), P)


@pytest.mark.parametrize("T,k,P", [(1, 1, 1), (1, 1, 2048), (9, 7, 63), (32, 2, 1025), (33, 31, 769), (64, 1, 64), (65, 16, 1024), (128, 16, 512),
                                   (341, 6, 384), (683, 3, 2048), (2048, 1, 2047)])
def test_reroute_permute_single_block_scan(ew, T, k, P):
    """One block: 6 to 16 waves whose totals the scan adds up, one to six slots per thread, one ranking wave up to all of them."""
    rng = np.random.default_rng(T + k + P)
    E = max(k, 8)
    ids = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)
    aid = rng.integers(0, 3, size=T).astype(np.int32)
    emap = rng.integers(0, P, size=(3, E)).astype(np.int32)
    emap[2, 0] = P - 1
    d = lambda a: torch.from_numpy(a).cuda()
    _check_permutation(ew.moe_reroute_permute(d(ids), d(aid), d(emap), 2, P), moe.reroute(ids, aid, emap), P)


def test_reroute_permute_all_to_one_slot_and_skip_inverse(ew):
    T, k, P = 3000, 4, 16
    ids = np.zeros((T, k), np.int32); aid = np.zeros(T, np.int32)
    emap = np.full((1, 1), 7, np.int32)
    slot, counts, offsets, por, rop = ew.moe_reroute_permute(torch.from_numpy(ids).cuda(), torch.from_numpy(aid).cuda(),
                                                             torch.from_numpy(emap).cuda(), 0, P, want_row_of_pair=False)
    assert rop is None and counts[7].item() == T * k and counts.sum().item() == T * k
    np.testing.assert_array_equal(por.cpu().numpy(), np.arange(T * k))


def test_empty_batch(ew):
    cfg = wl.get_config(1)
    _, emap = _expert_map(cfg)
    z = lambda *s: torch.zeros(s, dtype=torch.int32, device="cuda")
    slot, counts, offsets, por, rop = ew.moe_reroute_permute(z(0, 6), z(0), torch.from_numpy(emap).cuda(), cfg.N, cfg.P)
    assert counts.tolist() == [0] * cfg.P and offsets.tolist() == [0] * (cfg.P + 1)


@pytest.mark.parametrize("cfg_index,T", [(0, 64), (1, 64), (2, 300), (2, 341), (2, 342), (2, 2049), (2, 8192), (4, 256)])
def test_fused_route_reroute_permute(ew, cfg_index, T):
    cfg = wl.get_config(cfg_index)
    tuned, emap = _expert_map(cfg)
    rng = np.random.default_rng(cfg.seed)
    aid = wl.adapter_ids(cfg, T)
    logits = (rng.standard_normal((T, cfg.M)) * 0.9).astype(np.float32)
    if cfg.gate_bias:
        logits += wl.logit_bias_table(cfg, tuned)[aid]
    ids, w, *perm = ew.moe_route_reroute_permute(torch.from_numpy(logits).cuda(), torch.from_numpy(aid).cuda(),
                                                 torch.from_numpy(emap).cuda(), cfg.k, cfg.N, cfg.P)
    rids, rw = moe.route_topk(logits, cfg.k)
    np.testing.assert_array_equal(ids.cpu().numpy(), rids)
    np.testing.assert_allclose(w.cpu().numpy(), rw, rtol=2e-5, atol=1e-9)
    _check_permutation(perm, moe.reroute(rids, aid, emap), cfg.P)
    # same answer as the two stand-alone calls
    ids2, w2 = ew.moe_route_topk(torch.from_numpy(logits).cuda(), cfg.k)
    assert torch.equal(ids, ids2) and torch.equal(w, w2)


def test_c3_full_size(ew):
    """Config 3 at full size (1,048,576 tokens x top-6): every output bit-exact."""
    cfg = wl.get_config(3)
    tuned, emap = _expert_map(cfg)
    ids = wl.distinct_topk_ids(cfg)
    aid = wl.adapter_ids(cfg)
    got = ew.moe_reroute_permute(torch.from_numpy(ids).cuda(), torch.from_numpy(aid).cuda(),
                                 torch.from_numpy(emap).cuda(), cfg.N, cfg.P)
    torch.cuda.synchronize()
    _check_permutation(got, moe.reroute(ids, aid, emap), cfg.P)


@pytest.mark.parametrize("cfg_index,T", [(1, 64), (2, 8192), (3, 100000)])
def test_reroute_singleop_matches_fused(ew, cfg_index, T):
    """The unfused three-operator rerouting (paper Sec. 5.3 baseline) gives the oracle's slots bit for bit, and a
    permutation of those slots through an identity map equals the fused kernel's."""
    cfg = wl.get_config(cfg_index)
    tuned, emap = _expert_map(cfg)
    ids = wl.distinct_topk_ids(cfg, T)
    aid = wl.adapter_ids(cfg, T)
    d = lambda a: torch.from_numpy(a).cuda()
    slot = ew.moe_reroute_singleop(d(ids), d(aid), d(emap), cfg.N)
    ref = moe.reroute(ids, aid, emap)
    np.testing.assert_array_equal(slot.cpu().numpy(), ref)
    ident = torch.arange(cfg.P, dtype=torch.int32, device="cuda").reshape(1, cfg.P)
    zero = torch.zeros(T, dtype=torch.int32, device="cuda")
    two_step = ew.moe_reroute_permute(slot, zero, ident, 0, cfg.P)
    fused = ew.moe_reroute_permute(d(ids), d(aid), d(emap), cfg.N, cfg.P)
    for a, b in zip(two_step, fused):
        assert torch.equal(a, b)


def test_argument_errors(ew):
    z = torch.zeros((4, 2), dtype=torch.int32, device="cuda")
    a = torch.zeros(4, dtype=torch.int32, device="cuda")
    m = torch.zeros((1, 8), dtype=torch.int32, device="cuda")
    with pytest.raises(ew.EWError) as e:
        ew.moe_reroute_permute(z, a, m, 0, 5000)
    assert e.value.code == -6
    with pytest.raises(ew.EWError) as e:
        ew.moe_route_topk(torch.zeros((4, 8), device="cuda"), 9)
    assert e.value.code == -1
