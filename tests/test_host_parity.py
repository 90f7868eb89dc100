"""libtangram.so host integer calls vs the fp64 oracle, bit for bit (CPU only).

Covers Budget-Aware Clustering (Section 4.2.2), Budget Reservation and the
ragged per-group page tables (Eq. 4, Sections 4.1 and 4.2.1), Algorithm 1's
split map and the balanced partition plan, plus the error contract of
include/tangram.h.
"""
import ctypes
import json
import os

import numpy as np
import pytest
from hypothesis import given, settings, strategies as st

import oracle
from paper_2606_06302_amd import tangram as tg
from workloads import Geometry, config, free_list, pool_pages_for

GOLD = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "config1_hand.json")))


def _items_as_tuples(items):
    return [tuple(int(x) for x in it) for it in items.tolist()]


def _full_compare(geom, batch, ctx, ratio, budget, free, pool, grouping=0, mode=0, n_bins=7, split_target=33,
                  layers=None, bin_weights=None):
    L, H, Hp = geom.num_layers, geom.num_kv_heads, geom.heads_per_group
    G = H // Hp
    perm, gof, sof = tg.tg_cluster_heads(geom, budget, grouping)
    operm, ogof, osof = oracle.cluster_heads(budget, Hp, grouping)
    assert np.array_equal(perm, operm) and np.array_equal(gof, ogof) and np.array_equal(sof, osof)
    res = tg.tg_reserve(geom, ctx, ratio, budget, gof, free, pool)
    ores = oracle.reserve(ratio if ratio is not None else np.broadcast_to(budget, (batch, L, H)), ctx, ogof, G,
                          geom.page_size, free)
    assert np.array_equal(res["kv_len"], ores["kv_len"])
    assert np.array_equal(res["group_len"], ores["group_len"])
    assert np.array_equal(res["pt_offsets"], ores["offsets"])
    assert np.array_equal(res["pt_pages"], ores["pages"])
    assert res["pages_needed"] == ores["pages_needed"]
    for n_cta in (1, 8, 256, 1024):
        assert np.array_equal(tg.tg_split_map(geom, budget, perm, n_cta), oracle.split_map(budget, operm, Hp, n_cta))
    for layer in (range(L) if layers is None else layers):
        pl = tg.tg_build_plan(geom, batch, layer, res["kv_len"], res["pt_offsets"], gof, sof, mode, n_bins,
                              split_target, bin_weights=bin_weights)
        opl = oracle.partition_plan(ores["kv_len"], ores["offsets"], ogof, osof, layer, num_layers=L, num_groups=G,
                                    page_size=geom.page_size, mode=mode, n_bins=n_bins, split_target=split_target,
                                    bin_weights=bin_weights)
        assert _items_as_tuples(pl["items"]) == opl["items"]
        assert pl["bin_offsets"].tolist() == opl["bin_offsets"].tolist()
        assert np.array_equal(pl["unit_splits"], opl["unit_splits"])
        assert np.array_equal(pl["unit_partial_base"], opl["unit_partial_base"])
        assert pl["num_partials"] == opl["num_partials"]
    return res


def test_config1_matches_hand_values_and_oracle():
    wl = config(1)
    res = _full_compare(wl.geom, wl.batch, wl.ctx_len, wl.ratio, wl.budget, np.arange(100, dtype=np.int32), 100,
                        n_bins=8, split_target=16)
    assert res["pt_offsets"].tolist() == GOLD["offsets"]
    gof = tg.tg_cluster_heads(wl.geom, wl.budget)[1]
    pl = tg.tg_build_plan(wl.geom, 2, 0, res["kv_len"], res["pt_offsets"], gof,
                          tg.tg_cluster_heads(wl.geom, wl.budget)[2], 0, 8, 16)
    assert [list(t) for t in _items_as_tuples(pl["items"])] == GOLD["plan_split_target16_bins8"]["items"]
    fill = tg.tg_build_plan(wl.geom, 2, 0, res["kv_len"], res["pt_offsets"], gof,
                            tg.tg_cluster_heads(wl.geom, wl.budget)[2], tg.TG_PLAN_AOT_FILL, 8, 1)
    assert [list(t) for t in _items_as_tuples(fill["items"])] == GOLD["plan_fill_bins8"]["items"]
    assert fill["bin_offsets"].tolist() == GOLD["plan_fill_bins8"]["bin_offsets"]



def test_uniform_and_naive_plans_config1_hand():
    """The library's UNIFORM and NAIVE plans equal the hand-derived config-1 values."""
    from test_oracle_pins import uniform_gold_items
    wl = config(1)
    _, gof, sof = tg.tg_cluster_heads(wl.geom, wl.budget)
    res = tg.tg_reserve(wl.geom, wl.ctx_len, wl.ratio, None, gof, np.arange(100, dtype=np.int32), 100)
    gold = GOLD["plan_uniform_bins64"]
    u = tg.tg_build_plan(wl.geom, 2, 0, res["kv_len"], res["pt_offsets"], gof, sof, tg.TG_PLAN_UNIFORM, 64, 1)
    assert [list(t) for t in _items_as_tuples(u["items"])] == uniform_gold_items(gold)
    assert u["num_bins"] == gold["num_bins"] and u["bin_offsets"].tolist() == list(range(57))
    assert u["unit_splits"].tolist() == gold["unit_splits"] and u["num_partials"] == gold["num_partials"]
    assert u["unit_partial_base"].tolist() == gold["unit_partial_base"]
    gold = GOLD["plan_naive"]
    n = tg.tg_build_plan(wl.geom, 2, 0, res["kv_len"], res["pt_offsets"], gof, sof, tg.TG_PLAN_NAIVE, 64, 1)
    assert [list(t) for t in _items_as_tuples(n["items"])] == gold["items"]
    assert n["bin_offsets"].tolist() == gold["bin_offsets"] and n["num_partials"] == 0
    assert n["unit_partial_base"].tolist() == gold["unit_partial_base"]

@pytest.mark.parametrize("cfg", [1, 2, 4, 5])
def test_workload_configs_bit_exact(cfg):
    wl = config(cfg)
    gof = tg.tg_cluster_heads(wl.geom, wl.budget)[1]
    need = tg.tg_reserve(wl.geom, wl.ctx_len, wl.ratio, None, gof, np.zeros(0, np.int32), 0, size_query=True)
    pool = pool_pages_for(need["pages_needed"])
    free = free_list(wl, pool)
    for mode, nb, stg in [(0, 512, 2048), (1, 1, 1), (2, 512, 1), (3, 512, 1)]:
        _full_compare(wl.geom, wl.batch, wl.ctx_len, wl.ratio, wl.budget, free, pool, mode=mode, n_bins=nb,
                      split_target=stg)


@pytest.mark.slow
def test_config3_tables_and_two_layers_bit_exact():
    wl = config(3)
    gof = tg.tg_cluster_heads(wl.geom, wl.budget)[1]
    need = tg.tg_reserve(wl.geom, wl.ctx_len, wl.ratio, None, gof, np.zeros(0, np.int32), 0, size_query=True)
    pool = pool_pages_for(need["pages_needed"])
    _full_compare(wl.geom, wl.batch, wl.ctx_len, wl.ratio, wl.budget, free_list(wl, pool), pool, n_bins=512,
                  split_target=2048, layers=[0, 37])


@settings(max_examples=60, deadline=None)
@given(st.data())
def test_random_geometries_bit_exact(data):
    H = data.draw(st.sampled_from([1, 2, 3, 4, 6, 8, 12, 16]))
    Hp = data.draw(st.sampled_from([d for d in range(1, H + 1) if H % d == 0]))
    L = data.draw(st.integers(1, 3))
    B = data.draw(st.integers(1, 4))
    P = data.draw(st.sampled_from([1, 4, 16]))
    geom = Geometry(L, H, H * data.draw(st.integers(1, 3)), 8, P, Hp)
    grid = data.draw(st.booleans())
    shape = (L, H)
    rng = np.random.default_rng(data.draw(st.integers(0, 2**31)))
    if grid:   # ties and exact binary fractions
        budget = rng.integers(1, 9, size=shape) / 8.0
    else:
        budget = rng.uniform(1e-3, 1.0, size=shape)
    use_ratio = data.draw(st.booleans())
    ratio = np.clip(budget[None] + rng.uniform(-.03, .03, size=(B, L, H)), 0.02, 1.0) if use_ratio else None
    ctx = rng.integers(1, 500, size=B).astype(np.int32)
    grouping = data.draw(st.sampled_from([0, 1]))
    gof = tg.tg_cluster_heads(geom, budget, grouping)[1]
    need = tg.tg_reserve(geom, ctx, ratio, budget, gof, np.zeros(0, np.int32), 0, size_query=True)["pages_needed"]
    pool = need + int(rng.integers(0, 30))
    free = rng.permutation(pool).astype(np.int32)
    mode = data.draw(st.sampled_from([0, 1, 2, 3]))
    n_bins = data.draw(st.integers(1, 64))
    weights = None
    if mode == 3 and data.draw(st.booleans()):
        weights = rng.integers(1, data.draw(st.sampled_from([2, 1000, 65536])), size=n_bins).astype(np.int32)
    _full_compare(geom, B, ctx, ratio, budget, free, pool, grouping=grouping, mode=mode,
                  n_bins=n_bins, split_target=data.draw(st.integers(1, 300)), bin_weights=weights)


def test_fp64_ceil_pitfalls_match_oracle():
    geom = Geometry(1, 2, 2, 8, 16, 1)
    budget = np.array([[0.07, 0.29]])
    gof = tg.tg_cluster_heads(geom, budget)[1]
    res = tg.tg_reserve(geom, [100], None, budget, gof, np.arange(10, dtype=np.int32), 10)
    assert res["kv_len"].tolist() == [[[8, 29]]]


# ----------------------------------------------------------------- errors

def _geom1():
    return Geometry(1, 4, 8, 64, 16, 2)


@pytest.mark.parametrize("bad", [0.0, -1.0, 1.5, float("nan")])
def test_bad_budget_rejected(bad):
    b = np.array([[0.5, bad, 0.2, 0.1]])
    with pytest.raises(tg.TangramError) as e:
        tg.tg_cluster_heads(_geom1(), b)
    assert e.value.code == tg.TG_ERR_INVALID_ARG


def test_indivisible_groups_rejected():
    with pytest.raises(tg.TangramError) as e:
        tg.tg_cluster_heads(Geometry(1, 6, 6, 64, 16, 4), np.full((1, 6), .5))
    assert e.value.code == tg.TG_ERR_INVALID_ARG
    assert "heads_per_group" in tg.tg_last_error()


def test_out_of_pages_consumes_nothing():
    wl = config(1)
    gof = tg.tg_cluster_heads(wl.geom, wl.budget)[1]
    free = np.arange(79, dtype=np.int32)
    before = free.copy()
    with pytest.raises(tg.TangramError) as e:
        tg.tg_reserve(wl.geom, wl.ctx_len, wl.ratio, None, gof, free, 100)
    assert e.value.code == tg.TG_ERR_OUT_OF_PAGES and np.array_equal(free, before)


@pytest.mark.parametrize("free", [[0, 1, 1] + list(range(2, 90)), [-1] + list(range(1, 90)), list(range(80)) + [200]])
def test_bad_page_ids_rejected(free):
    wl = config(1)
    gof = tg.tg_cluster_heads(wl.geom, wl.budget)[1]
    free = np.array(free, dtype=np.int32)
    if free[-1] == 200:        # an out-of-pool id that is consumed
        free = np.concatenate([[200], np.arange(79)]).astype(np.int32)
    with pytest.raises(tg.TangramError) as e:
        tg.tg_reserve(wl.geom, wl.ctx_len, wl.ratio, None, gof, free, 100)
    assert e.value.code == tg.TG_ERR_INVALID_ARG


@pytest.mark.parametrize("threads", ["1", "4", "8"])
def test_page_id_check_across_host_threads(threads, monkeypatch):
    """600 000 consumed pages, so the id check runs on several host threads, each marking its chunk of the
    list in a bitmap of its own: a repeat inside one chunk, a repeat across two chunks and an id outside the
    pool must all be rejected, and a valid permutation must be taken as is."""
    monkeypatch.setenv("TG_HOST_THREADS", threads)
    geom = Geometry(1, 1, 1, 64, 16, 1)
    n = 600_000
    ctx, ratio = np.array([16 * n], np.int32), np.ones((1, 1, 1))
    gof = np.zeros((1, 1), np.int32)
    pool = n + 5000
    free = np.random.default_rng(5).permutation(pool).astype(np.int32)
    res = tg.tg_reserve(geom, ctx, ratio, None, gof, free, pool)
    assert res["pages_needed"] == n and np.array_equal(res["pt_pages"], free[:n])
    for i, j in ((3, 7), (5, n - 2), (n // 2 - 1, n // 2 + 1)):
        bad = free.copy()
        bad[j] = bad[i]
        with pytest.raises(tg.TangramError) as e:
            tg.tg_reserve(geom, ctx, ratio, None, gof, bad, pool)
        assert e.value.code == tg.TG_ERR_INVALID_ARG and "twice" in tg.tg_last_error(), (i, j)
    ok = free.copy()
    ok[n] = ok[0]              # a repeat beyond the consumed prefix is never examined
    assert np.array_equal(tg.tg_reserve(geom, ctx, ratio, None, gof, ok, pool)["pt_pages"], free[:n])
    out = free.copy()
    out[n - 1] = pool
    with pytest.raises(tg.TangramError) as e:
        tg.tg_reserve(geom, ctx, ratio, None, gof, out, pool)
    assert e.value.code == tg.TG_ERR_INVALID_ARG and "outside the pool" in tg.tg_last_error()


def test_plan_rejects_length_beyond_table():
    wl = config(1)
    perm, gof, sof = tg.tg_cluster_heads(wl.geom, wl.budget)
    res = tg.tg_reserve(wl.geom, wl.ctx_len, wl.ratio, None, gof, np.arange(100, dtype=np.int32), 100)
    kv = res["kv_len"].copy()
    kv[0, 0, 2] = 129        # head 2's group holds 8 pages = 128 rows
    with pytest.raises(tg.TangramError) as e:
        tg.tg_build_plan(wl.geom, 2, 0, kv, res["pt_offsets"], gof, sof, 0, 8, 16)
    assert e.value.code == tg.TG_ERR_INVALID_ARG


def test_status_strings_and_version():
    assert tg.tg_status_string(0) == "ok"
    assert tg.tg_status_string(tg.TG_ERR_OUT_OF_PAGES) == "out of pages"
    assert tg.tg_status_string(tg.TG_ERR_NO_MEMORY) == "out of host memory"
    assert tg.tg_version() >> 16 == 1


@pytest.mark.parametrize("cfg", [2, 4, 5])
def test_prefill_schedule_bit_exact_on_configs(cfg):
    wl = config(cfg)
    gof = tg.tg_cluster_heads(wl.geom, wl.budget)[1]
    res = tg.tg_reserve(wl.geom, wl.ctx_len, wl.ratio, None, gof, np.zeros(0, np.int32), 0, size_query=True)
    C = wl.chunk_len or 512
    for n_xcd in (8, 3, 1):
        got = tg.tg_prefill_schedule(wl.geom, wl.batch, C, 0, res["kv_len"], n_xcd)
        ref, _ = oracle.prefill_schedule(res["kv_len"], 0, C, wl.geom.gqa, n_xcd)
        assert got.tolist() == ref.tolist()


@settings(max_examples=40, deadline=None)
@given(st.data())
def test_prefill_schedule_random_bit_exact(data):
    H = data.draw(st.sampled_from([1, 2, 4, 8]))
    gqa = data.draw(st.integers(1, 16))
    L = data.draw(st.integers(1, 3))
    B = data.draw(st.integers(1, 5))
    C = data.draw(st.integers(1, 1200))
    n_xcd = data.draw(st.integers(1, 12))
    layer = data.draw(st.integers(0, L - 1))
    rng = np.random.default_rng(data.draw(st.integers(0, 2**31)))
    kv = rng.integers(0, data.draw(st.sampled_from([1, 70, 3000])), size=(B, L, H)).astype(np.int32)
    geom = Geometry(L, H, H * gqa, 128, 16, 1)
    got = tg.tg_prefill_schedule(geom, B, C, layer, kv, n_xcd)
    ref, _ = oracle.prefill_schedule(kv, layer, C, gqa, n_xcd)
    assert got.tolist() == ref.tolist()


def test_prefill_schedule_of_many_blocks():
    """More blocks than the binding's first call has room for."""
    kv = np.random.default_rng(3).integers(0, 5000, (40, 1, 8)).astype(np.int32)
    got = tg.tg_prefill_schedule(Geometry(1, 8, 128, 64, 16, 2), 40, 300, 0, kv)
    ref, _ = oracle.prefill_schedule(kv, 0, 300, 16, 8)
    assert len(got) > 4096 and np.array_equal(got, ref)


def test_prefill_schedule_errors():
    geom = Geometry(1, 2, 4, 128, 16, 1)
    kv = np.ones((1, 1, 2), np.int32)
    for bad in [dict(n_xcd=0), dict(n_xcd=65)]:
        with pytest.raises(tg.TangramError):
            tg.tg_prefill_schedule(geom, 1, 8, 0, kv, **bad)
    with pytest.raises(tg.TangramError):
        tg.tg_prefill_schedule(geom, 1, 0, 0, kv)
    with pytest.raises(tg.TangramError):
        tg.tg_prefill_schedule(geom, 1, 8, 1, kv)


def test_weighted_fill_config3_layer_bit_exact_and_errors():
    wl = config(3)
    gof = tg.tg_cluster_heads(wl.geom, wl.budget)[1]
    need = tg.tg_reserve(wl.geom, wl.ctx_len, wl.ratio, None, gof, np.zeros(0, np.int32), 0, size_query=True)
    pool = pool_pages_for(need["pages_needed"])
    w = np.where((np.arange(1024) // 4) % 8 % 2 == 1, 955, 1044).astype(np.int32)
    _full_compare(wl.geom, wl.batch, wl.ctx_len, wl.ratio, wl.budget, free_list(wl, pool), pool, mode=3,
                  n_bins=1024, split_target=1, layers=[5], bin_weights=w)
    geom = Geometry(1, 2, 4, 128, 16, 1)
    kv = np.full((1, 1, 2), 40, np.int32)
    off = np.array([0, 3, 6], np.int64)
    gof1, sof1 = np.array([[0, 1]], np.int32), np.zeros((1, 2), np.int32)
    for bad, mode in [([0, 1], 3), ([1, 65536], 3), ([1, 1], 0)]:
        with pytest.raises(tg.TangramError):
            tg.tg_build_plan(geom, 1, 0, kv, off, gof1, sof1, mode, 2, 4, bin_weights=np.array(bad, np.int32))


# ------------------------------------------- compression fused into prefill

def _compress_compare(geom, batch, ctx, ratio, budget, sel_ratio, starts, toks, C, R, layers=None):
    L, H, Hp = geom.num_layers, geom.num_kv_heads, geom.heads_per_group
    G = H // Hp
    perm, gof, sof = tg.tg_cluster_heads(geom, budget)
    res = tg.tg_reserve(geom, ctx, ratio, budget, gof, np.arange(10**6, dtype=np.int32), 10**6)
    for layer in (range(L) if layers is None else layers):
        pl = tg.tg_compress_plan(geom, batch, layer, C, starts, toks, sel_ratio, budget, res["kv_len"],
                                 res["pt_offsets"], gof, sof, R)
        sr = sel_ratio if sel_ratio is not None else np.broadcast_to(budget, (batch, L, H))
        items, cur, cnt = oracle.compress_plan(sr, res["kv_len"], starts, toks, res["pt_offsets"], gof, sof, layer,
                                               num_layers=L, num_groups=G, rows_per_item=R)
        assert _items_as_tuples(pl["items"]) == items
        assert np.array_equal(pl["write_begin"], cur) and np.array_equal(pl["keep_count"], cnt)
    return res


def test_compress_plan_config5_chunk_after_history_bit_exact():
    """Config 5's chunk (512 tokens after a 16384-token history), reserved for the whole 16896-token context."""
    wl = config(5)
    C = wl.chunk_len
    starts = wl.ctx_len
    _compress_compare(wl.geom, wl.batch, wl.ctx_len + C, wl.ratio, wl.budget, wl.ratio, starts,
                      np.full(wl.batch, C), C, 64)


@settings(max_examples=60, deadline=None)
@given(st.data())
def test_compress_plan_random_bit_exact(data):
    H = data.draw(st.sampled_from([1, 2, 4, 8]))
    Hp = data.draw(st.sampled_from([h for h in (1, 2, 4, 8) if H % h == 0]))
    L = data.draw(st.integers(1, 3))
    P = data.draw(st.sampled_from([1, 3, 16]))
    B = data.draw(st.integers(1, 5))
    geom = Geometry(L, H, H, 64, P, Hp)
    rng = np.random.default_rng(data.draw(st.integers(0, 2**31)))
    budget = rng.uniform(0.01, 1.0, size=(L, H))
    ratio = np.clip(budget[None] + rng.uniform(-0.05, 0.05, size=(B, L, H)), 0.01, 1.0)
    ctx = rng.integers(1, 3000, size=B).astype(np.int32)
    C = int(rng.integers(1, 700))
    starts = np.array([int(rng.integers(0, c + 1)) for c in ctx], dtype=np.int32)
    toks = np.minimum(C, np.maximum(0, ctx - starts + rng.integers(-3, 50, size=B))).astype(np.int32)
    choice = data.draw(st.sampled_from(["same", "overflow", "budget"]))
    sel = {"same": ratio, "overflow": np.minimum(1.0, ratio * 1.7), "budget": None}[choice]
    R = data.draw(st.sampled_from([1, 5, 64, 256]))
    _compress_compare(geom, B, ctx, ratio, budget, sel, starts, toks, C, R)


def test_compress_plan_fp64_pitfall_and_size_query():
    geom = Geometry(1, 1, 1, 64, 16, 1)
    budget = np.array([[0.07]])
    res = tg.tg_reserve(geom, [100], None, budget, [[0]], np.arange(10, dtype=np.int32), 10)
    assert res["kv_len"][0, 0, 0] == 8
    got = [tg.tg_compress_plan(geom, 1, 0, 50, [c0], [50], None, budget, res["kv_len"], res["pt_offsets"], [[0]],
                               [[0]], 3) for c0 in (0, 50)]
    assert [(int(p["write_begin"][0, 0]), int(p["keep_count"][0, 0])) for p in got] == [(0, 4), (4, 4)]
    assert [p["num_items"] for p in got] == [2, 2]


def test_compress_plan_errors():
    geom = Geometry(1, 2, 2, 64, 16, 2)
    budget = np.array([[0.5, 0.25]])
    res = tg.tg_reserve(geom, [64], None, budget, [[0, 0]], np.arange(10, dtype=np.int32), 10)
    kv, off = res["kv_len"], res["pt_offsets"]
    ok = dict(chunk_start=[0], chunk_tokens=[32], ratio=None, budget=budget, kv_len=kv, pt_offsets=off,
              group_of=[[0, 0]], slot_of=[[0, 1]])

    def call(C=32, R=64, layer=0, **kw):
        a = dict(ok, **kw)
        return tg.tg_compress_plan(geom, 1, layer, C, a["chunk_start"], a["chunk_tokens"], a["ratio"], a["budget"],
                                   a["kv_len"], a["pt_offsets"], a["group_of"], a["slot_of"], R)

    assert call()["num_items"] == 2
    for kw in (dict(C=0), dict(C=tg.TG_COMPRESS_MAX_CHUNK + 1), dict(R=0), dict(R=tg.TG_COMPRESS_MAX_ROWS + 1),
               dict(layer=1), dict(chunk_start=[-1]), dict(chunk_tokens=[33]), dict(chunk_tokens=[-1]),
               dict(chunk_start=[2**31 - 10]), dict(ratio=np.array([[[0.5, 1.5]]])), dict(ratio=np.array([[[0.0, 0.5]]])),
               dict(slot_of=[[0, 2]]), dict(group_of=[[0, 1]]), dict(kv_len=kv + 100), dict(kv_len=kv * 0 - 1)):
        with pytest.raises(tg.TangramError) as e:
            call(**kw)
        assert e.value.code == tg.TG_ERR_INVALID_ARG, kw


def test_compress_launch_validation_on_host():
    """tg_compress rejects unsupported shapes before touching the device; an empty plan enqueues nothing."""
    g = Geometry(1, 2, 2, 128, 16, 2)

    def args(**kw):
        a = dict(geom=g, batch=1, chunk_len=8, dtype=tg.TG_BF16, num_items=0)
        a.update(kw)
        return tg.tg_compress_args(tg._geom(a["geom"]), a["batch"], a["chunk_len"], a["dtype"], None, None, None,
                                   None, None, None, a["num_items"], None, None, None)

    tg.tg_compress(args())                       # nothing to do: OK without a device
    for kw, code in ((dict(dtype=7), tg.TG_ERR_UNSUPPORTED), (dict(geom=Geometry(1, 2, 2, 96, 16, 2)),
                                                              tg.TG_ERR_UNSUPPORTED),
                     (dict(chunk_len=0), tg.TG_ERR_INVALID_ARG), (dict(chunk_len=tg.TG_COMPRESS_MAX_CHUNK + 1),
                                                                  tg.TG_ERR_INVALID_ARG),
                     (dict(batch=0), tg.TG_ERR_INVALID_ARG), (dict(num_items=-1), tg.TG_ERR_INVALID_ARG),
                     (dict(num_items=3), tg.TG_ERR_INVALID_ARG), (dict(geom=Geometry(1, 3, 3, 128, 16, 2)),
                                                                 tg.TG_ERR_INVALID_ARG)):
        with pytest.raises(tg.TangramError) as e:
            tg.tg_compress(args(**kw))
        assert e.value.code == code, kw


# ------------------------------------------------ memory footprint of paging

@pytest.mark.parametrize("cfg", [1, 2, 4, 5])
def test_footprint_configs_bit_exact(cfg):
    wl = config(cfg)
    g = wl.geom
    for Hp in (1, 2, 4, 8):
        if g.num_kv_heads % Hp:
            continue
        geom = Geometry(g.num_layers, g.num_kv_heads, g.num_q_heads, g.head_dim, g.page_size, Hp)
        for grouping in (tg.TG_GROUP_CLUSTERED, tg.TG_GROUP_ADJACENT):
            _, gof, _ = tg.tg_cluster_heads(geom, wl.budget, grouping)
            got = tg.tg_memory_footprint(geom, wl.ctx_len, wl.ratio, None, gof)
            ref = oracle.memory_footprint(wl.ratio, wl.ctx_len, gof, g.num_kv_heads // Hp, Hp, g.page_size)
            assert got == ref, (cfg, Hp, grouping)
            need = tg.tg_reserve(geom, wl.ctx_len, wl.ratio, None, gof, np.zeros(0, np.int32), 0,
                                 size_query=True)["pages_needed"]
            assert got["ragged_pages"] == need


def test_footprint_budget_broadcast_and_errors():
    geom = Geometry(1, 4, 4, 64, 16, 2)
    budget = np.array([[0.1, 1.0, 0.1, 1.0]])
    _, gof, _ = tg.tg_cluster_heads(geom, budget)
    f = tg.tg_memory_footprint(geom, [160], None, budget, gof)
    assert (f["ragged_slots"], f["monolithic_slots"], f["full_slots"], f["retained_slots"]) == (352, 640, 640, 352)
    for args in (([0], None, budget, gof), ([160], None, np.array([[0.1, 1.5, 0.1, 1.0]]), gof),
                 ([160], None, budget, np.array([[0, 1, 2, 0]])), ([160], None, None, gof)):
        with pytest.raises(tg.TangramError) as e:
            tg.tg_memory_footprint(geom, *args)
        assert e.value.code == tg.TG_ERR_INVALID_ARG


# ------------------------------------------------ decode steps: headroom, open-ended plans

@settings(max_examples=40, deadline=None)
@given(st.data())
def test_headroom_and_open_plans_bit_exact(data):
    H = data.draw(st.sampled_from([2, 4, 8]))
    Hp = data.draw(st.sampled_from([h for h in (1, 2, 4) if H % h == 0]))
    L = data.draw(st.integers(1, 3))
    P = data.draw(st.sampled_from([1, 5, 16]))
    B = data.draw(st.integers(1, 5))
    geom = Geometry(L, H, 2 * H, 64, P, Hp)
    rng = np.random.default_rng(data.draw(st.integers(0, 2**31)))
    budget = rng.uniform(0.01, 1.0, size=(L, H))
    ratio = np.clip(budget[None] + rng.uniform(-0.05, 0.05, size=(B, L, H)), 0.01, 1.0)
    ctx = rng.integers(1, 2000, size=B).astype(np.int32)
    headroom = rng.integers(0, 300, size=B).astype(np.int32)
    _, gof, sof = tg.tg_cluster_heads(geom, budget)
    res = tg.tg_reserve(geom, ctx, ratio, None, gof, np.arange(10**6, dtype=np.int32), 10**6, headroom=headroom)
    ores = oracle.reserve(ratio, ctx, gof, H // Hp, P, np.arange(10**6), headroom=headroom)
    assert np.array_equal(res["pt_offsets"], ores["offsets"]) and np.array_equal(res["kv_len"], ores["kv_len"])
    mode = data.draw(st.sampled_from([tg.TG_PLAN_AOT, tg.TG_PLAN_NAIVE, tg.TG_PLAN_UNIFORM, tg.TG_PLAN_AOT_FILL]))
    layer = data.draw(st.integers(0, L - 1))
    pl = tg.tg_build_plan(geom, B, layer, res["kv_len"], res["pt_offsets"], gof, sof, mode | tg.TG_PLAN_OPEN_END,
                          7, 29)
    opl = oracle.partition_plan(ores["kv_len"], ores["offsets"], gof, sof, layer, num_layers=L, num_groups=H // Hp,
                                page_size=P, mode=mode, n_bins=7, split_target=29, open_end=True)
    assert _items_as_tuples(pl["items"]) == opl["items"]
    assert pl["bin_offsets"].tolist() == opl["bin_offsets"].tolist()
    assert sum(1 for it in opl["items"] if it[5] < 0) == B * H


def test_headroom_config1_hand_and_errors():
    wl = config(1)
    _, gof, _ = tg.tg_cluster_heads(wl.geom, wl.budget)
    res = tg.tg_reserve(wl.geom, wl.ctx_len, wl.ratio, None, gof, np.arange(100, dtype=np.int32), 100,
                        headroom=[20, 20])
    assert res["pt_offsets"].tolist() == [0, 10, 44, 54, 88]
    with pytest.raises(tg.TangramError) as e:
        tg.tg_reserve(wl.geom, wl.ctx_len, wl.ratio, None, gof, np.arange(100, dtype=np.int32), 100,
                      headroom=[0, -1])
    assert e.value.code == tg.TG_ERR_INVALID_ARG
    with pytest.raises(tg.TangramError) as e:
        tg.tg_build_plan(wl.geom, 2, 0, res["kv_len"], res["pt_offsets"], gof, gof, 0x200)
    assert e.value.code == tg.TG_ERR_INVALID_ARG


def test_append_launch_validation_on_host():
    g = Geometry(1, 2, 2, 128, 16, 2)
    bad = tg.tg_append_args(tg._geom(Geometry(1, 2, 2, 96, 16, 2)), 1, 0, tg.TG_BF16, *([None] * 8), None)
    with pytest.raises(tg.TangramError) as e:
        tg.tg_append(bad)
    assert e.value.code == tg.TG_ERR_UNSUPPORTED
    for kw in (dict(layer=1), dict(batch=0), dict(layer=0)):   # the last: NULL device pointers
        a = dict(batch=1, layer=0)
        a.update(kw)
        args = tg.tg_append_args(tg._geom(g), a["batch"], a["layer"], tg.TG_BF16, *([None] * 8), None)
        with pytest.raises(tg.TangramError) as e:
            tg.tg_append(args)
        assert e.value.code == tg.TG_ERR_INVALID_ARG, kw


def test_decode_append_arguments_checked_on_host():
    """tg_decode's in-launch append needs both token arrays and the live lengths; the call is refused on
    the host, before any launch (the device pointers below are never dereferenced)."""
    g = Geometry(1, 2, 4, 128, 16, 2)
    fake = 1 << 20

    def args(**kw):
        a = tg.make_decode_args(g, 1, tg.TG_BF16, None, None, None, None, None, 4, 1, None, None, 0, None)
        for f in ("q", "kv_pool", "pt_pages", "items", "bin_offsets", "out"):
            setattr(a, f, fake)
        for k, v in kw.items():
            setattr(a, k, v)
        return a

    for kw in (dict(append_k=fake), dict(append_v=fake), dict(append_k=fake, append_v=fake),
               dict(append_k=fake, live_len=fake)):
        with pytest.raises(tg.TangramError) as e:
            tg.tg_decode(args(**kw))
        assert e.value.code == tg.TG_ERR_INVALID_ARG, kw


def test_misaligned_device_buffers_refused_on_host():
    """The device calls move Q, K, V, tokens, outputs and pool rows with 16-byte accesses: a buffer that is
    not 16-byte aligned is refused with TG_ERR_INVALID_ARG before anything is enqueued (the fake device
    pointers below are never dereferenced)."""
    g = Geometry(1, 2, 4, 128, 16, 2)
    fake, off = 1 << 20, (1 << 20) + 8

    def refused(fn, args, field):
        setattr(args, field, off)
        rc = fn(ctypes.byref(args), None)
        assert rc == tg.TG_ERR_INVALID_ARG and b"16-byte aligned" in tg._lib.tg_last_error(), field
        setattr(args, field, fake)

    d = tg.make_decode_args(g, 1, tg.TG_BF16, None, None, None, None, None, 4, 1, None, None, 0, None)
    for f in ("q", "kv_pool", "pt_pages", "items", "bin_offsets", "out"):
        setattr(d, f, fake)
    for f in ("q", "kv_pool", "out"):
        refused(tg._lib.tg_decode, d, f)
    d.append_k, d.append_v, d.live_len = fake, fake, fake
    for f in ("append_k", "append_v"):
        refused(tg._lib.tg_decode, d, f)

    pre = tg.tg_prefill_args(tg._geom(g), 1, 1, 0, tg.TG_BF16, *([fake] * 10))
    for f in ("q", "k_new", "v_new", "kv_pool", "out"):
        refused(tg._lib.tg_prefill, pre, f)

    cmp = tg.tg_compress_args(tg._geom(g), 1, 8, tg.TG_BF16, fake, fake, fake, fake, fake, fake, 1, fake, fake,
                              fake)
    for f in ("k_new", "v_new", "kv_pool"):
        refused(tg._lib.tg_compress, cmp, f)

    app = tg.tg_append_args(tg._geom(g), 1, 0, tg.TG_BF16, *([fake] * 9))
    for f in ("k_tok", "v_tok", "kv_pool"):
        refused(tg._lib.tg_append, app, f)


def test_read_probe_slab_sizes_checked_on_host():
    """tg_read_probe runs only the 2, 4 and 8 KiB slab kernels: every other slab size is refused before
    anything is enqueued, and an accepted size goes on to the remaining argument checks (here a zero
    worker count), so nothing is launched either way."""
    def call(d, dtype, page_size=16, n_workers=0):
        g = tg._geom(Geometry(1, 2, 2, d, page_size, 2))
        return tg._lib.tg_read_probe(ctypes.byref(g), dtype, None, None, None, 0, n_workers, None, None)

    for d, dtype in ((32, tg.TG_BF16), (96, tg.TG_BF16), (160, tg.TG_BF16), (48, tg.TG_F32), (80, tg.TG_F32),
                     (112, tg.TG_F32), (256, tg.TG_F32), (512, tg.TG_BF16), (8, tg.TG_F32)):
        assert call(d, dtype) == tg.TG_ERR_UNSUPPORTED, (d, dtype)      # 1, 3, 5, 3, 5, 7, 16, 16 KiB, 512 B
    for d, dtype in ((64, tg.TG_BF16), (128, tg.TG_BF16), (256, tg.TG_BF16), (32, tg.TG_F32), (64, tg.TG_F32),
                     (128, tg.TG_F32)):
        assert call(d, dtype) == tg.TG_ERR_INVALID_ARG, (d, dtype)      # 2, 4, 8 KiB: on to n_workers
    assert call(128, tg.TG_BF16, page_size=8) == tg.TG_ERR_INVALID_ARG  # 8 rows of 256 B = 2 KiB
    assert call(128, tg.TG_BF16, page_size=12) == tg.TG_ERR_UNSUPPORTED


@settings(max_examples=40, deadline=None)
@given(st.data())
def test_split_map_plan_bit_exact(data):
    H = data.draw(st.sampled_from([2, 4, 8]))
    Hp = data.draw(st.sampled_from([h for h in (1, 2, 4, 8) if H % h == 0]))
    L = data.draw(st.integers(1, 3))
    P = data.draw(st.sampled_from([1, 16]))
    B = data.draw(st.integers(1, 6))
    geom = Geometry(L, H, H, 64, P, Hp)
    rng = np.random.default_rng(data.draw(st.integers(0, 2**31)))
    budget = rng.uniform(0.01, 1.0, size=(L, H))
    ratio = np.clip(budget[None] + rng.uniform(-0.05, 0.05, size=(B, L, H)), 0.01, 1.0)
    ctx = rng.integers(1, 3000, size=B).astype(np.int32)
    perm, gof, sof = tg.tg_cluster_heads(geom, budget)
    res = tg.tg_reserve(geom, ctx, ratio, None, gof, np.arange(10**6, dtype=np.int32), 10**6)
    n_cta = data.draw(st.sampled_from([1, 7, 256, 1024]))
    S = tg.tg_split_map(geom, budget, perm, n_cta)
    flag = data.draw(st.sampled_from([0, tg.TG_PLAN_OPEN_END]))
    for layer in range(L):
        pl = tg.tg_build_plan(geom, B, layer, res["kv_len"], res["pt_offsets"], gof, sof,
                              tg.TG_PLAN_SPLIT_MAP | flag, 1, 1, bin_weights=S[layer])
        opl = oracle.partition_plan(res["kv_len"], res["pt_offsets"], gof, sof, layer, num_layers=L,
                                    num_groups=H // Hp, page_size=P, mode=oracle.MODE_SPLIT_MAP, bin_weights=S[layer],
                                    open_end=bool(flag))
        assert _items_as_tuples(pl["items"]) == opl["items"]
        assert pl["bin_offsets"].tolist() == opl["bin_offsets"].tolist()
        assert np.array_equal(pl["unit_splits"], opl["unit_splits"])
        assert np.array_equal(pl["unit_partial_base"], opl["unit_partial_base"])
        assert pl["num_bins"] == int(S[layer].sum())
    with pytest.raises(tg.TangramError):
        tg.tg_build_plan(geom, B, 0, res["kv_len"], res["pt_offsets"], gof, sof, tg.TG_PLAN_SPLIT_MAP, 1, 1)


# ------------------------------------------------ calibration and request lifecycle

@settings(max_examples=40, deadline=None)
@given(st.data())
def test_implicit_ratios_and_budget_bit_exact(data):
    rng = np.random.default_rng(data.draw(st.integers(0, 2**31)))
    L, H, N = data.draw(st.integers(1, 3)), data.draw(st.integers(1, 8)), data.draw(st.integers(1, 60))
    S = data.draw(st.integers(1, 5))
    rho = data.draw(st.sampled_from([0.05, 0.3, 0.5, 0.7, 1.0, float(rng.uniform(0.01, 1.0))]))
    samples = []
    for _ in range(S):
        sc = (rng.integers(-6, 7, size=(L, H, N)) / 2).astype(np.float32)       # many ties
        sc[rng.random(sc.shape) < 0.05] = np.nan
        sc[rng.random(sc.shape) < 0.05] = -0.0
        r, c = tg.tg_implicit_ratios(sc, rho)
        orr, oc = oracle.implicit_ratios(sc, rho)
        assert np.array_equal(c, oc) and np.array_equal(r, orr)
        samples.append(r)
    alpha = data.draw(st.sampled_from([0.0, 1.0, 2.0, 3.5]))
    B = tg.tg_calibrate_budget(np.stack(samples), alpha, 1e-3)
    assert np.array_equal(B, oracle.calibrate_budget(np.stack(samples), alpha, 1e-3))


def test_calibration_errors():
    for args in ((np.zeros((1, 1, 4), np.float32), 0.0), (np.zeros((1, 1, 4), np.float32), 1.5)):
        with pytest.raises(tg.TangramError):
            tg.tg_implicit_ratios(*args)
    for kw in (dict(alpha=-1.0), dict(floor=0.0), dict(floor=1.5)):
        with pytest.raises(tg.TangramError):
            tg.tg_calibrate_budget(np.full((2, 1, 1), 0.5), **kw)
    with pytest.raises(tg.TangramError):
        tg.tg_calibrate_budget(np.full((2, 1, 1), 1.5))


@pytest.mark.parametrize("cfg", [1, 2, 4])
def test_release_and_concat_bit_exact(cfg):
    wl = config(cfg)
    g = wl.geom
    _, gof, _ = tg.tg_cluster_heads(g, wl.budget)
    pool = 10**7
    res = tg.tg_reserve(g, wl.ctx_len, wl.ratio, None, gof, free_list(wl, pool), pool)
    rng = np.random.default_rng(cfg)
    fin = rng.random(wl.batch) < 0.4
    freed, off, pages = tg.tg_release_requests(g, res["pt_offsets"], res["pt_pages"], fin)
    of, oo, op = oracle.release_requests(res["pt_offsets"], res["pt_pages"], fin, g.num_layers, g.num_groups)
    assert np.array_equal(freed, of) and np.array_equal(off, oo) and np.array_equal(pages, op)
    # readmit the finished requests from the freed pages and append their tables
    if fin.any():
        again = tg.tg_reserve(g, wl.ctx_len[fin], wl.ratio[fin], None, gof, freed, pool)
        o2, p2 = tg.tg_concat_tables(g, off, pages, again["pt_offsets"], again["pt_pages"])
        e2, q2 = oracle.concat_tables(off, pages, again["pt_offsets"], again["pt_pages"])
        assert np.array_equal(o2, e2) and np.array_equal(p2, q2)
        assert sorted(p2.tolist()) == sorted(res["pt_pages"].tolist())


@pytest.mark.parametrize("dtype,d,gqa,n_bins,want", [
    (tg.TG_BF16, 128, 8, 1, 1), (tg.TG_BF16, 128, 8, 256, 1), (tg.TG_BF16, 128, 8, 257, 2), (tg.TG_BF16, 128, 1, 512, 2),
    (tg.TG_BF16, 128, 16, 768, 3), (tg.TG_BF16, 128, 8, 769, 4), (tg.TG_BF16, 128, 8, 2 ** 31 - 1, 4),
    (tg.TG_BF16, 64, 1, 1792, 1), (tg.TG_BF16, 64, 4, 384, 1), (tg.TG_BF16, 64, 4, 385, 2), (tg.TG_BF16, 64, 5, 200, 1),
    (tg.TG_BF16, 64, 5, 1024, 4), (tg.TG_F32, 64, 2, 1024, 1), (tg.TG_F32, 128, 16, 1024, 1)])
def test_bins_per_decode_workgroup(dtype, d, gqa, n_bins, want):
    """One to four bins per workgroup where every wave runs its own (bf16 matrix kernel, by plan size), else one: the
    mapping from bins to workgroups, and so to XCDs, that weights and time stamps are grouped by."""
    assert tg.tg_decode_bins_per_workgroup(Geometry(1, 2, 2 * gqa, d, 16, 2), dtype, n_bins) == want


def test_bins_per_decode_workgroup_refuses():
    for geom, dtype, n_bins in ((Geometry(1, 2, 2, 128, 16, 2), tg.TG_BF16, 0), (Geometry(1, 2, 2, 96, 16, 2), tg.TG_BF16, 8),
                                (Geometry(1, 2, 34, 128, 16, 2), tg.TG_BF16, 8), (Geometry(1, 2, 2, 128, 16, 2), 7, 8)):
        with pytest.raises(tg.TangramError):
            tg.tg_decode_bins_per_workgroup(geom, dtype, n_bins)


@pytest.mark.parametrize("d,B,H,gqa,C,hist,pays", [
    (128, 1, 8, 4, 512, 13000, True),       # one request, a long history
    (128, 16, 8, 4, 512, 4000, False),      # blocks enough, of one length
    (64, 1, 8, 4, 512, 13000, True),
    (64, 25, 8, 1, 408, 5000, True),        # 400 blocks one per CU, two rounds of them: cut at head_dim 64
    (64, 20, 8, 1, 37, 350, False),         # short blocks: the merge costs more
    (128, 7, 2, 16, 266, 13000, False),     # 17 row tiles a piece: three pieces on one XCD's 32 CUs
    (128, 7, 2, 16, 120, 13000, True),      # 8 row tiles: they fit
    (96, 1, 8, 4, 512, 13000, False),       # no such kernel
])
def test_prefill_split_pays(d, B, H, gqa, C, hist, pays):
    """The choice between whole blocks and the key-split launch: a quarter of the KV heads keep all of the history, the
    others an eighth."""
    keep = np.where(np.arange(H) % 4 == 0, hist, hist // 8)
    kv = np.ascontiguousarray(np.broadcast_to(keep, (B, 1, H))).astype(np.int32)
    assert tg.tg_prefill_split_pays(Geometry(1, H, H * gqa, d, 16, 1), B, C, 0, kv) == pays


def test_prefill_split_pays_up_to_512_units():
    kv = np.full((65, 1, 8), 300, np.int32)
    kv[0, 0, 0] = 9000
    g = Geometry(1, 8, 8, 128, 16, 1)
    assert tg.tg_prefill_split_pays(g, 64, 5, 0, kv[:64]) and not tg.tg_prefill_split_pays(g, 65, 5, 0, kv)


def test_prefill_split_pays_refuses():
    g, kv = Geometry(1, 2, 4, 128, 16, 1), np.full((1, 1, 2), 100, np.int32)
    for args in ((g, 0, 8, 0, kv), (g, 1, 0, 0, kv), (g, 1, 8, 1, kv), (g, 1, 8, 0, -kv)):
        with pytest.raises(tg.TangramError):
            tg.tg_prefill_split_pays(*args)
