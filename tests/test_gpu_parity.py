"""GPU parity: every stage of the library against the CPU oracle on the same seeded inputs.

Integer results (selected experts, slots, offsets, permutation) must be bit-exact; floating point
results must be within max|gpu - ref| / max|ref| <= 1e-2 (bf16) / 1e-4 (fp32)."""
import numpy as np
import pytest
import torch

import synth
from oracle import revive_oracle as orc
from harness import GpuLayer, TOL, compare_selection, f64, rel_err

pytestmark = pytest.mark.gpu


def _i(t):
    return t.cpu().numpy()


def _small(name, **kw):
    return synth.scaled(synth.get_config(name), **kw)


# reduced variants whose full oracle runs in seconds but which still span several row tiles of
# 256 (bf16) / 64 (fp32) with ragged tails, several 1024-row dispatch chunks and empty slots
SMALL = {
    "c1": synth.get_config("c1"),
    "c1_big": _small("c1", T=700),
    "c2s": _small("c2", T=1500, H=512, I=320, I_shared=192),
    "c2m": _small("c2", T=1500, H=512, I=320, I_shared=192, E=16, k=4, n_ranks=4, slots_per_rank=5,
                  failed_ranks=(2,), n_unprotected=-1),
    "c3s": _small("c3", T=900, H=512, I=256, I_shared=256),
    "c4s": _small("c4", T=900, H=512, I=256, I_shared=256),
    "c5s": _small("c5", T=1100, H=448, I=192, I_shared=128),
    # shortest reduction dimensions the bf16 GEMM accepts (2 and 4 K-steps of 32): pipeline prologue and tail only
    "k64": _small("c2", T=700, H=64, I=64, I_shared=64, E=16, k=2, n_ranks=4, slots_per_rank=5, failed_ranks=(1,),
                  n_unprotected=-1),
    "k128": _small("c2", T=600, H=128, I=64, I_shared=128, E=16, k=3, n_ranks=4, slots_per_rank=5, failed_ranks=(),
                   n_unprotected=-1),
    # uneven expert load (router columns scaled by exp(0.6 z)): slots with no rows next to slots of many row-tiles
    "c2_skew": _small("c2", T=1500, H=512, I=320, I_shared=192, router_skew=0.6),
    "c3_skew": _small("c3", T=900, H=512, I=256, I_shared=256, router_skew=0.6),
    # the largest expert count, slot count, top-k and group count the library accepts; ranks 3 and 4 are neighbours,
    # so rank 4's primaries lose both copies (8 lost experts), rank 40 only degrades
    "max": _small("c3", T=300, H=128, I=64, I_shared=64, E=512, k=32, n_ranks=64, slots_per_rank=16, max_replicas=2,
                  n_group=32, topk_group=8, failed_ranks=(3, 4, 40), n_unprotected=-1),
}


@pytest.fixture(scope="module", params=list(SMALL))
def small_layer(request):
    torch.manual_seed(0)
    g = GpuLayer(SMALL[request.param])
    yield g
    g.close()


def test_map_tables_match_oracle(small_layer):
    g = small_layer
    table, count, alive = g.layer.get_map()
    m = g.oracle_map()
    assert np.array_equal(table, m.l2p_table) and np.array_equal(count, m.l2p_count)
    assert np.array_equal(alive, m.slot_alive)
    assert g.stats == dict(n_live_slots=m.n_live_slots, n_live_experts=m.n_live_experts,
                           n_lost_experts=m.n_lost_experts, n_degraded_experts=m.n_degraded_experts)


def test_route_on_given_logits_is_bit_exact(small_layer):
    g = small_layer
    c = g.cfg
    logits = synth.draw_logits(c, g.device)
    _, top_l, top_w, top_p = g.layer.route(None, None, c.T, logits=logits, logits_given=True)
    m = g.oracle_map()
    s = orc.scores(f64(logits), c.score_fn)
    sel = orc.masked_selection_scores(s, m.l2p_count)
    ref_l = orc.select_topk(sel, c.k, c.n_group, c.topk_group)
    assert np.array_equal(_i(top_l), ref_l)
    assert np.array_equal(_i(top_p), orc.remap(ref_l, m))
    assert np.abs(f64(top_w) - orc.gate_weights(s, ref_l)).max() < 2e-7
    assert m.l2p_count[_i(top_l)].min() > 0                      # never a masked expert


def test_router_logits_and_near_ties(small_layer):
    g = small_layer
    c = g.cfg
    lg, top_l, top_w, top_p = g.layer.route(g.x, g.w_router_packed, c.T)
    ref_lg = orc.router_logits(f64(g.x), f64(g.w_router))
    assert rel_err(f64(lg), ref_lg) < (1e-5 if c.dtype == "fp32" else 1e-5)
    m = g.oracle_map()
    # selection from the GPU's own logits: exact
    s_gpu = orc.scores(f64(lg), c.score_fn)
    ref_from_gpu = orc.select_topk(orc.masked_selection_scores(s_gpu, m.l2p_count), c.k, c.n_group, c.topk_group)
    assert np.array_equal(_i(top_l), ref_from_gpu)
    # selection from the oracle's fp64 logits: may differ only on near-ties (gap < 1e-5)
    s = orc.scores(ref_lg, c.score_fn)
    sel = orc.masked_selection_scores(s, m.l2p_count)
    ref = orc.select_topk(sel, c.k, c.n_group, c.topk_group)
    near, bad = compare_selection(c, _i(top_l), sel, ref)
    print(f"[{c.name}] near-ties: {len(near)} of {c.T} tokens, mismatches: {len(bad)}")
    assert not bad


def test_dispatch_is_bit_exact(small_layer):
    g = small_layer
    c = g.cfg
    logits = synth.draw_logits(c, g.device)
    _, top_l, top_w, top_p = g.layer.route(None, None, c.T, logits=logits, logits_given=True)
    x_perm, offs, dst, src = g.layer.dispatch(g.x, top_p, c.T)
    ref_offs, ref_dst, ref_src = orc.dispatch_indices(_i(top_p), c.P)
    assert np.array_equal(_i(offs), ref_offs)
    assert np.array_equal(_i(dst), ref_dst)
    assert np.array_equal(_i(src), ref_src)
    assert torch.equal(x_perm, g.x[torch.from_numpy(ref_src // c.k).to(g.device).long()])
    S = c.slots_per_rank
    counts = np.diff(_i(offs))
    for r in np.nonzero(g.failed)[0]:
        assert counts[r * S:(r + 1) * S].sum() == 0            # a failed rank receives nothing
    # determinism: a second call gives identical indices
    _, offs2, dst2, src2 = g.layer.dispatch(g.x, top_p, c.T)
    assert torch.equal(dst, dst2) and torch.equal(src, src2) and torch.equal(offs, offs2)


def _experts_f64(g):
    return {e: g.expert_f64(e) for e in range(g.cfg.E)}


def test_layer_against_oracle(small_layer):
    """Whole layer; the oracle is fed the GPU's logits so that the routing is identical and every
    intermediate can be compared element by element."""
    g = small_layer
    c = g.cfg
    r = g.forward()
    tr = orc.layer_staged(f64(g.x), None, _experts_f64(g), g.shared_f64(), g.p2l, g.oracle_map(), c.k, c.score_fn,
                          c.n_group, c.topk_group, logits=f64(r["logits"]))
    assert np.array_equal(_i(r["topk_logical"]), tr.topk_logical)
    assert np.array_equal(_i(r["topk_phys"]), tr.topk_phys)
    assert np.array_equal(_i(r["slot_offsets"]), tr.slot_offsets)
    assert np.array_equal(_i(r["dst_row"]), tr.dst_row) and np.array_equal(_i(r["src_of"]), tr.src_of)
    assert np.array_equal(f64(r["x_perm"]), tr.x_perm)
    tol = TOL[c.dtype]
    errs = {"y_perm": rel_err(f64(r["y_perm"]), tr.y_perm), "out": rel_err(f64(r["out"]), tr.out)}
    if tr.y_shared is not None:
        errs["y_shared"] = rel_err(f64(r["y_shared"]), tr.y_shared)
    print(f"[{c.name}] rel errors: " + ", ".join(f"{k}={v:.2e}" for k, v in errs.items()))
    for k, v in errs.items():
        assert v < tol, (k, v)
    # and against the definition of the layer (dense gate matrix over all experts), own fp64 logits
    if c.T <= 128:
        dense = orc.layer_definition(f64(g.x), f64(g.w_router), _experts_f64(g), g.shared_f64(),
                                     g.oracle_map().l2p_count, c.k, c.score_fn, c.n_group, c.topk_group)
        assert rel_err(f64(r["out"]), dense) < tol


def test_no_failure_and_pure_remap_outputs():
    """Sec. 3.4: as long as every expert keeps a replica the output is the unfailed layer's."""
    cfg = SMALL["c3s"]
    g = GpuLayer(cfg, failed=[])
    try:
        base = g.forward()
        out0 = base["out"].clone()
        top0 = base["topk_logical"].clone()
        phys0 = base["topk_phys"].clone()
        stats = g.set_failed(cfg.failed_ranks)
        assert stats["n_lost_experts"] == 0 and stats["n_degraded_experts"] > 0
        r = g.forward()
        assert torch.equal(r["topk_logical"], top0)
        assert not torch.equal(r["topk_phys"], phys0)
        S = cfg.slots_per_rank
        alive_rows = np.diff(_i(r["slot_offsets"]))
        for f in cfg.failed_ranks:
            assert alive_rows[f * S:(f + 1) * S].sum() == 0
        same = torch.equal(r["out"], out0)
        err = rel_err(f64(r["out"]), f64(out0))
        print(f"pure remap: bit-identical={same}, rel diff={err:.2e}")
        assert err < 1e-6 if not same else True
    finally:
        g.close()


def test_fewer_tokens_than_the_context_was_sized_for():
    """A context created for T_max tokens serves any T <= T_max (decode batches shrink and grow)."""
    cfg = SMALL["c2m"]
    g = GpuLayer(cfg)
    try:
        experts = _experts_f64(g)
        for T in (cfg.T, 257, 64, 1, cfg.T):
            L = g.layer
            lg, top_l, top_w, top_p = L.route(g.x, g.w_router_packed, T)
            x_perm, offs, dst, src = L.dispatch(g.x, top_p, T)
            y_perm, y_sh = L.expert_ffn(x_perm, offs, T, x=g.x, w_sh_gate_up=g.sh_gate_up, w_sh_down=g.sh_down)
            out = L.combine(y_perm, dst, top_w, y_sh, T)
            tr = orc.layer_staged(f64(g.x[:T]), None, experts, g.shared_f64(), g.p2l, g.oracle_map(), cfg.k,
                                  cfg.score_fn, cfg.n_group, cfg.topk_group, logits=f64(lg))
            assert np.array_equal(_i(top_p), tr.topk_phys) and np.array_equal(_i(dst), tr.dst_row)
            assert _i(offs)[-1] == T * cfg.k
            assert rel_err(f64(out), tr.out) < TOL[cfg.dtype], T
        with pytest.raises(Exception):
            g.layer.route(g.x, g.w_router_packed, cfg.T + 1)
    finally:
        g.close()


def test_update_map_rejects_and_keeps_tables():
    cfg = SMALL["c1"]
    g = GpuLayer(cfg, with_weights=False)
    try:
        before = g.layer.get_map()
        bad = np.ones(cfg.n_ranks, np.uint8)
        assert g.layer.update_map_status(bad) == -4
        bad[:] = 0
        bad[1] = 3
        assert g.layer.update_map_status(bad) == -1
        after = g.layer.get_map()
        assert all(np.array_equal(a, b) for a, b in zip(before, after))
        logits = synth.draw_logits(cfg, g.device)
        _, top_l, _, top_p = g.layer.route(None, None, cfg.T, logits=logits, logits_given=True)
        m = g.oracle_map()
        assert m.slot_alive[_i(top_p)].all()
    finally:
        g.close()


def test_empty_and_single_token():
    cfg = SMALL["c2s"]
    g = GpuLayer(cfg)
    try:
        L = g.layer
        # T = 0: offsets all zero, nothing else touched
        x_perm, offs, dst, src = L.dispatch(g.x, torch.zeros(0, cfg.k, dtype=torch.int32, device=g.device), 0)
        assert _i(offs).tolist() == [0] * (cfg.P + 1)
        # T = 1
        lg, top_l, top_w, top_p = L.route(g.x, g.w_router_packed, 1)
        x_perm, offs, dst, src = L.dispatch(g.x, top_p, 1)
        y_perm, y_sh = L.expert_ffn(x_perm, offs, 1, x=g.x, w_sh_gate_up=g.sh_gate_up, w_sh_down=g.sh_down)
        out = L.combine(y_perm, dst, top_w, y_sh, 1)
        experts = {int(e): g.expert_f64(int(e)) for e in _i(top_l).ravel()}
        tr = orc.layer_staged(f64(g.x[:1]), None, experts, g.shared_f64(), g.p2l, g.oracle_map(), cfg.k, cfg.score_fn,
                              cfg.n_group, cfg.topk_group, logits=f64(lg[:1]))
        assert np.array_equal(_i(dst)[:cfg.k], tr.dst_row)
        assert rel_err(f64(out[:1]), tr.out) < TOL[cfg.dtype]
    finally:
        g.close()


def test_graph_replay_matches_eager_across_mask_flips():
    """One captured graph, replayed after map updates: same executable, results equal to the eager
    calls and to the oracle under the map in force (Sec. 3.6: no recompilation on recovery)."""
    cfg = SMALL["c5s"]
    g = GpuLayer(cfg, failed=[])
    try:
        experts = _experts_f64(g)
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            g.forward(stream=stream)
            stream.synchronize()
            g.capture(stream)
            exec_id = g.layer.graph_exec_id(g.graph)
            for failed in ([], list(cfg.failed_ranks), [0], []):
                g.set_failed(failed, stream=stream)
                for rep in range(3):
                    g.buf["out"].zero_()
                    g.replay(stream)
                    stream.synchronize()
                    out_graph = g.buf["out"].clone()
                    tr = orc.layer_staged(f64(g.x), None, experts, g.shared_f64(), g.p2l, g.oracle_map(), cfg.k,
                                          cfg.score_fn, logits=f64(g.buf["logits"]))
                    assert np.array_equal(_i(g.buf["topk_phys"]), tr.topk_phys)
                    assert np.array_equal(_i(g.buf["dst_row"]), tr.dst_row)
                    assert rel_err(f64(out_graph), tr.out) < TOL[cfg.dtype]
                    g.forward(stream=stream)          # the program's own eager work between replays
                    stream.synchronize()
                    assert torch.equal(g.buf["out"], out_graph)
                assert g.layer.graph_exec_id(g.graph) == exec_id
    finally:
        g.close()


@pytest.mark.parametrize("name", ["c2m", "c1_big"])
def test_every_token_picks_the_same_experts(name):
    """Degenerate routing: identical logits rows send all T tokens to the same k experts, so a few
    slots receive T rows each (many row-tiles in one group, every other slot empty, one-bin
    histograms in the dispatch) and ties between equal logits go to the lower expert id."""
    cfg = SMALL[name]
    g = GpuLayer(cfg)
    try:
        E = cfg.E
        row = torch.zeros(E, dtype=torch.float32)
        row[: E // 2] = 1.0                       # a tie among the first half, a tie among the second
        logits = row.repeat(cfg.T, 1).to(g.device)
        r = g.forward(logits=logits)
        tr = orc.layer_staged(f64(g.x), None, _experts_f64(g), g.shared_f64(), g.p2l, g.oracle_map(), cfg.k, cfg.score_fn,
                              cfg.n_group, cfg.topk_group, logits=f64(logits))
        live = np.nonzero(g.oracle_map().l2p_count > 0)[0]
        assert np.array_equal(_i(r["topk_logical"])[0], live[: cfg.k])      # lowest live ids win the ties
        assert np.array_equal(_i(r["topk_logical"]), tr.topk_logical)
        assert np.abs(f64(r["topk_weight"]) - 1.0 / cfg.k).max() < 1e-6
        assert np.array_equal(_i(r["topk_phys"]), tr.topk_phys)
        assert np.array_equal(_i(r["slot_offsets"]), tr.slot_offsets)
        assert np.array_equal(_i(r["dst_row"]), tr.dst_row) and np.array_equal(_i(r["src_of"]), tr.src_of)
        counts = np.diff(tr.slot_offsets)
        assert counts.max() >= cfg.T // cfg.max_replicas and (counts == 0).sum() >= cfg.P - cfg.k * cfg.max_replicas
        assert rel_err(f64(r["out"]), tr.out) < TOL[cfg.dtype]
    finally:
        g.close()


def test_out_of_range_slot_ids_drop_the_row():
    """Boundary behaviour of the ABI, not of the method: a slot id outside [0, P) in a caller's
    topk_phys drops that routed row: it takes no place in the sort (dst_row = -1) and the combine
    skips it.  The kept rows sort as if the dropped ones were absent."""
    cfg = SMALL["c2m"]
    g = GpuLayer(cfg)
    try:
        L, T, k, P, H = g.layer, cfg.T, cfg.k, cfg.P, cfg.H
        rng = np.random.default_rng(3)
        phys = rng.integers(0, P, size=(T, k)).astype(np.int32)
        bad = rng.random((T, k)) < 0.05
        phys[bad] = np.where(rng.random(bad.sum()) < 0.5, -1, P + 7)
        d_phys = torch.from_numpy(phys).to(g.device)
        x_perm, offs, dst, src = L.dispatch(g.x, d_phys, T)
        flat, keep = phys.ravel(), ~bad.ravel()
        kept = np.nonzero(keep)[0]
        ref_offs, ref_dst_kept, ref_src_kept = orc.dispatch_indices(flat[kept], P)   # the oracle on the kept rows alone
        ref_dst = np.full(T * k, -1, dtype=np.int32)
        ref_dst[kept] = ref_dst_kept
        n = kept.size
        assert np.array_equal(_i(offs), ref_offs) and _i(offs)[-1] == n
        assert np.array_equal(_i(dst), ref_dst)
        assert np.array_equal(_i(src)[:n], kept[ref_src_kept])
        assert torch.equal(x_perm[:n], g.x[torch.from_numpy(kept[ref_src_kept] // k).to(g.device)])
        # combine: only the kept rows contribute
        y_perm = g.x.new_zeros(T * k, H)
        y_perm[:n] = torch.randn(n, H, device=g.device).to(y_perm.dtype)
        w = torch.rand(T, k, device=g.device, dtype=torch.float32)
        out = L.combine(y_perm, dst, w, None, T)
        yp, ww = f64(y_perm), f64(w)
        ref = np.zeros((T, H))
        for t in range(T):
            for j in range(k):
                d = ref_dst[t * k + j]
                if d >= 0:
                    ref[t] += ww[t, j] * yp[d]
        assert rel_err(f64(out), ref) < TOL[cfg.dtype]
    finally:
        g.close()


def test_data_path_calls_refuse_bad_arguments_without_launching():
    """Error behaviour of the boundary: wrong sizes, missing state and null pointers come back as a
    status with a message; nothing is launched and the context stays usable."""
    import ctypes as C
    from paper_2602_21140_amd.binding import ReviveError, ReviveLayer, lib
    cfg = SMALL["c2m"]
    L = ReviveLayer(cfg)
    try:
        T = cfg.T
        x = synth.draw_x(cfg, L.device)
        w_r = synth.draw_router(cfg, L.device).t().contiguous()
        with pytest.raises(ReviveError) as e:          # no map yet
            L.route(x, w_r, T)
        assert e.value.status == -3
        L.set_placement(synth.make_placement(cfg))
        L.update_map(synth.failed_mask(cfg))
        with pytest.raises(ReviveError) as e:          # more tokens than the context was sized for
            L.route(x, w_r, T + 1)
        assert e.value.status == -1 and "T_max" in str(e.value)
        raw = lib()
        null = C.c_void_p(None)
        i32 = L.empty(T, cfg.k, dtype=torch.int32)
        f32 = L.empty(T, cfg.k, dtype=torch.float32)
        lg = L.empty(T, cfg.E, dtype=torch.float32)
        rc = raw.revive_route(L._ctx, null, null, lg.data_ptr(), 0, T, i32.data_ptr(), f32.data_ptr(), i32.data_ptr(), null)
        assert rc == -1                                  # x and w_router missing although logits are not given
        rc = raw.revive_dispatch(L._ctx, x.data_ptr(), i32.data_ptr(), T, null, null, null, null, null)
        assert rc == -1
        rc = raw.revive_combine(L._ctx, null, null, null, null, T, null, null)
        assert rc == -1
        assert raw.revive_last_error(L._ctx).decode() != ""
        # the context still works
        _, top_l, top_w, top_p = L.route(x, w_r, T)
        assert int(top_p.min()) >= 0
    finally:
        L.close()


def test_random_sequence_of_map_updates_under_one_graph():
    """Sec. 3.6: recovery, further failures and add-backs are table updates under one captured graph.
    A random sequence of failure sets (rank failures and single-expert failures), some applied
    several in a row without a step in between, some refused because too few experts would stay
    reachable: after every accepted update the replay matches the oracle under the map in force,
    after every refused one the previous map is still in force."""
    cfg = SMALL["c4s"]
    g = GpuLayer(cfg, failed=[])
    try:
        experts = _experts_f64(g)
        rng = np.random.default_rng(11)
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            g.forward(stream=stream)
            stream.synchronize()
            g.capture(stream)
            exec_id = g.layer.graph_exec_id(g.graph)
            in_force = (synth.failed_mask(cfg, []), None)
            accepted = refused = 0
            for step in range(40):
                for _ in range(int(rng.integers(1, 4))):          # one to three updates before the next step
                    n_fail = int(rng.choice([0, 1, 2, 3, 6, 12, 24, 30, 31, cfg.n_ranks]))
                    ranks = synth.failed_mask(cfg, rng.choice(cfg.n_ranks, size=n_fail, replace=False))
                    ef = (rng.random(cfg.E) < 0.05).astype(np.uint8) if rng.random() < 0.5 else None
                    m = orc.build_map(g.p2l, ranks, cfg.slots_per_rank, cfg.E, cfg.max_replicas, expert_failed=ef)
                    ok = orc.enough_live_experts(m.l2p_count, cfg.k, cfg.n_group, cfg.topk_group)
                    if ok:
                        g.set_failed(np.nonzero(ranks)[0], stream=stream, expert_failed=ef)
                        in_force = (ranks, ef)
                        accepted += 1
                    else:
                        with pytest.raises(Exception):
                            g.layer.update_map(ranks, stream=stream, expert_failed=ef)
                        refused += 1
                g.buf["out"].zero_()
                g.replay(stream)
                stream.synchronize()
                m = orc.build_map(g.p2l, in_force[0], cfg.slots_per_rank, cfg.E, cfg.max_replicas, expert_failed=in_force[1])
                table, count, alive = g.layer.get_map()
                assert np.array_equal(count, m.l2p_count) and np.array_equal(table, m.l2p_table)
                tr = orc.layer_staged(f64(g.x), None, experts, g.shared_f64(), g.p2l, m, cfg.k, cfg.score_fn,
                                      cfg.n_group, cfg.topk_group, logits=f64(g.buf["logits"]))
                assert np.array_equal(_i(g.buf["topk_logical"]), tr.topk_logical), step
                assert np.array_equal(_i(g.buf["topk_phys"]), tr.topk_phys), step
                assert np.array_equal(_i(g.buf["dst_row"]), tr.dst_row), step
                assert rel_err(f64(g.buf["out"]), tr.out) < TOL[cfg.dtype], step
            assert g.layer.graph_exec_id(g.graph) == exec_id
            print(f"map updates accepted {accepted}, refused {refused}")
            assert accepted > 20 and refused > 0
    finally:
        g.close()


@pytest.mark.parametrize("name", ["c2m", "c4s"])
def test_a_masked_expert_with_a_towering_logit_leaves_the_weights_finite(name):
    """Sec. 3.4 "Missing experts": a masked expert takes no part in the selection, whatever its logit.
    Here every lost expert's logit towers a thousand above all live ones (reachable through given
    logits): the chosen experts and their weights must be those of the live experts alone."""
    cfg = SMALL[name]
    g = GpuLayer(cfg, with_weights=False)
    try:
        m = g.oracle_map()
        lost = np.nonzero(m.l2p_count == 0)[0]
        assert lost.size > 0
        logits = synth.draw_logits(cfg, g.device)
        logits[:, torch.from_numpy(lost).to(g.device)] += 1000.0
        _, top_l, top_w, top_p = g.layer.route(None, None, cfg.T, logits=logits, logits_given=True)
        lg = f64(logits)
        live = np.nonzero(m.l2p_count > 0)[0]
        if cfg.score_fn == "softmax":      # the oracle's softmax over all logits underflows to 0/0 here: restrict it to the live ones,
            s = np.zeros_like(lg)          # which gives the same selection and the same renormalised weights
            s[:, live] = orc.scores(lg[:, live], "softmax")
        else:
            s = orc.scores(lg, cfg.score_fn)
        ref_l = orc.select_topk(orc.masked_selection_scores(s, m.l2p_count), cfg.k, cfg.n_group, cfg.topk_group)
        assert np.array_equal(_i(top_l), ref_l)
        w = f64(top_w)
        assert np.isfinite(w).all()
        assert np.abs(w - orc.gate_weights(s, ref_l)).max() < 2e-7
        assert np.abs(w.sum(axis=1) - 1.0).max() < 1e-6
        assert np.array_equal(_i(top_p), orc.remap(ref_l, m))
    finally:
        g.close()


@pytest.mark.parametrize("raw", [True, False])  # False: a torch without the private function for it
def test_calls_without_a_stream_take_the_current_one(raw, monkeypatch):
    from paper_2602_21140_amd import ReviveLayer, binding

    if not raw:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
        monkeypatch.setattr(binding, "_raw_stream", None)
    side = torch.cuda.Stream()
    assert ReviveLayer._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert ReviveLayer._stream(None) == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert ReviveLayer._stream(side) == side.cuda_stream and ReviveLayer._stream(None) != side.cuda_stream
