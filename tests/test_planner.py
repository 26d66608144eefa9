"""Host-side tests of the C-ABI library: planner tables bit-exact against an
independent derivation, tile lists cover the work exactly once, error paths,
exported symbols.  No GPU needed (lora_plan_create is pure host code)."""
import collections
import ctypes
import heapq
import os
import re

import numpy as np
import pytest
from hypothesis import given, settings, strategies as st

from oracle import plan_ref
from paper_2411_00915_amd import autotune, binding as B
from paper_2411_00915_amd import device, workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _export(w, variant=B.LORA_VARIANT_AUTO):
    p = device.make_plan(w, variant)
    v = B.lora_plan_export(p)
    q = B.lora_plan_query(p)
    p.destroy()
    return v, q


def _check_tables(w, v):
    tok, perm, ga, go = plan_ref.tables(w.T, w.seg_indptr, w.seg_adapter, w.adapter_rank)
    assert v["num_tokens"] == w.T
    assert np.array_equal(v["token_adapter"], tok)
    assert np.array_equal(v["perm"], perm)
    assert np.array_equal(v["group_adapter"], ga)
    assert np.array_equal(v["group_offset"], go)
    return tok, perm


def _check_gemm_tables(w, v, tok, perm):
    """the fused forward's row order and adapter stages: a permutation, and every tile's stages cover the columns of
    exactly the adapters its rows carry, once each (the order of rows and stages is the planner's choice)"""
    if v["kernel_family"] != B.LORA_VARIANT_TILED:
        return
    if w.T == 0:
        assert v["gemm_order"].shape[0] == 0 and v["gemm_stage"].shape[0] == 0
        return
    assert v["gemm_order"].shape[0] == w.T
    plan_ref.check_gemm_tables(w.T, tok, w.adapter_rank, v["gemm_order"], v["gemm_stage_offset"], v["gemm_stage"],
                               stage_cols=64)


def _check_tiles(w, v, tok, perm):
    both = v["kernel_family"] == B.LORA_VARIANT_TILED
    assert both or v["expand_tiles"].shape[0] == 0
    if v["shrink_kernel_family"] != B.LORA_VARIANT_TILED:          # (it is TILED whenever kernel_family is)
        assert not both and v["shrink_tiles"].shape[0] == 0
        return
    max_r = int(w.adapter_rank.max()) if w.num_adapters else 0
    P = v["v_parts"]
    assert P in (1, 2, 4)
    et_ = [(t[0], t[1], t[2], t[3], t[4]) for t in v["expand_tiles"]]
    if len(perm):
        for part in range(P):          # every K part covers the (token, rank) plane exactly once
            st_ = [(t[0], t[1], t[2], t[3], t[4]) for t in v["shrink_tiles"] if (t[5] >> 8) & 15 == part]
            plan_ref.check_cover(st_, tok, perm, max(max_r, 1), adapter_rank=w.adapter_rank, rank_axis=True)
        assert all((t[5] >> 12) & 15 == P and (t[5] >> 8) & 15 < P for t in v["shrink_tiles"])
        if both:
            plan_ref.check_cover(et_, tok, perm, w.N)
    else:
        assert v["shrink_tiles"].shape[0] == 0 and not et_
    for t in v["shrink_tiles"]:
        tb, jb = t[5] & 15, (t[5] >> 4) & 15
        assert t[2] <= 16 * tb and t[4] <= 16 * jb and tb in (1, 2, 4, 8) and 1 <= jb <= 8
        assert t[3] % 16 == 0
    for t in v["expand_tiles"]:
        tb = t[5] & 15
        assert t[2] <= 16 * tb and tb in (1, 2, 4, 8) and t[3] % 64 == 0


def _check_mixture(w, m, variant=B.LORA_VARIANT_AUTO):
    """Mixture mode: the plan must be the plan of the tokens' own branches (merged adapter's segments without
    adapter) plus a second batch, over exactly the tokens that are not the merged adapter's, all on that adapter."""
    p = device.make_plan(w, variant, merged_adapter=m)
    v = B.lora_plan_export(p)
    R, v_bytes, ws_bytes = B.lora_plan_query(p)
    p.destroy()
    if m < 0 or m >= w.num_adapters or w.adapter_rank[m] == 0:
        assert v["merged_adapter"] == -1 and v["num_unmerge"] == 0 and v["unmerge_v_offset"] == 0
        tok, perm = _check_tables(w, v)
        _check_tiles(w, v, tok, perm)
        return v
    own_seg, removal = plan_ref.mixture_tables(w.T, w.seg_indptr, w.seg_adapter, w.adapter_rank, m)
    own = wl.Workload(w.name, w.dtype, w.T, w.K, w.N, w.seg_indptr, own_seg, w.adapter_rank, w.adapter_scale, w.x, None)
    tok, perm = _check_tables(own, v)
    _check_tiles(own, v, tok, perm)
    assert v["merged_adapter"] == m
    assert np.array_equal(v["unmerge_perm"], np.nonzero(removal)[0])
    # the removal's tiles: every (token, rank index of m) and every (token, feature) exactly once
    rem_tok = np.where(removal, m, -1)
    rperm = v["unmerge_perm"]
    P2 = v["unmerge_v_parts"]
    if len(rperm) and v["unmerge_shrink_tiles"].shape[0]:
        for part in range(P2):
            st_ = [(t[0], t[1], t[2], t[3], t[4]) for t in v["unmerge_shrink_tiles"] if (t[5] >> 8) & 15 == part]
            plan_ref.check_cover(st_, rem_tok, rperm, int(w.adapter_rank[m]), adapter_rank=w.adapter_rank, rank_axis=True)
        plan_ref.check_cover([(t[0], t[1], t[2], t[3], t[4]) for t in v["unmerge_expand_tiles"]], rem_tok, rperm, w.N)
    # v: own parts, then (256-byte aligned) the removal's
    own_bytes = v["v_parts"] * w.T * R * 4
    assert v["unmerge_v_offset"] == (own_bytes + 255) // 256 * 256
    assert v_bytes == v["unmerge_v_offset"] + P2 * w.T * v["unmerge_v_row_stride"] * 4
    assert ws_bytes >= v_bytes + 2 * w.T * (R + v["unmerge_v_row_stride"]) * 2 and ws_bytes % 256 == 0
    if v["gemm_order"].shape[0]:
        plan_ref.check_gemm_tables(w.T, tok, w.adapter_rank, v["gemm_order"], v["gemm_stage_offset"], v["gemm_stage"],
                                   stage_cols=64, merged=m, removal=removal)
    return v


@pytest.mark.parametrize("name,m", [("cfg2", 5), ("cfg3", 1), ("cfg4", 0), ("cfg4", 77), ("cfg1", 2)])
def test_mixture_mode_tables(name, m):
    w = wl.CONFIGS[name](with_w=False)
    v = _check_mixture(w, m)
    assert v["num_unmerge"] == w.T - int(np.sum(plan_ref.tables(w.T, w.seg_indptr, w.seg_adapter, w.adapter_rank)[0] == m))
    if name == "cfg3":
        # 3 of the 4 requests need the removal; the tiles of the merged adapter's 1024 tokens carry no stage at all
        assert v["num_unmerge"] == 3072 and v["num_active"] == 3072
        off = v["gemm_stage_offset"]
        assert sum(1 for t in range(len(off) - 1) if off[t] == off[t + 1]) == 4


@settings(max_examples=100, deadline=None)
@given(st.lists(st.tuples(st.integers(0, 40), st.integers(-1, 5)), min_size=0, max_size=20),
       st.lists(st.sampled_from([0, 8, 16, 32, 64, 128]), min_size=6, max_size=6),
       st.integers(0, 5), st.sampled_from([64, 1000]))
def test_random_mixture_tables(segs, ranks, m, N):
    lengths = [s[0] for s in segs]
    T = sum(lengths)
    indptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32) if segs else np.zeros(1, np.int32)
    w = wl.Workload("h", "bf16", T, 64, N, indptr, np.asarray([s[1] for s in segs], np.int32), np.asarray(ranks, np.int32),
                    np.ones(6, np.float32), np.zeros((T, 64), np.float32), None)
    _check_mixture(w, m, B.LORA_VARIANT_TILED)


@pytest.mark.parametrize("m", [-1, 2])
@pytest.mark.parametrize("lengths,n_a,ranks", [
    ([400] + [2] * 60, 61, (64, 16)),                    # one long request, many short ones; a short last segment
    ([63, 64, 65, 1, 127] * 3, 15, (8, 128)),            # around the 64 rows of a segment
    ([17] * 30, 30, (32,)), ([40] * 19, 19, (16, 128)),  # what has no room in one piece
    ([500, 2, 2, 1], 4, (64,)), ([5] * 12, 3, (8,)),     # two segments; no more than one
    ([64] * 8, 8, (32,))])                               # nothing to gain: stays sorted
def test_rows_of_the_fused_gemm_are_dealt_to_wavefronts(lengths, n_a, ranks, m):
    """Every 64 rows hold each of their adapters as one run (a wavefront adds a delta per run), and neither the sum over the tiles of the longest wavefront nor the longest of all is above the sorted order's."""
    lengths = np.asarray(lengths + [9, 30], np.int32)    # (and requests without adapter)
    ads = np.concatenate([np.arange(len(lengths) - 2) % n_a, [-1, -1]]).astype(np.int32)
    rank = np.asarray([ranks[a % len(ranks)] for a in range(n_a)], np.int32)
    T = int(lengths.sum())
    w = wl.Workload("h", "bf16", T, 64, 640, np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32), ads, rank,
                    np.ones(n_a, np.float32), np.zeros((T, 64), np.float32), None)
    v = _check_mixture(w, m, B.LORA_VARIANT_TILED)
    if m < 0:
        _check_gemm_tables(w, v, v["token_adapter"], v["perm"])
    tok, order = v["token_adapter"], v["gemm_order"]
    carries = (tok >= 0) | (np.repeat(ads, lengths) != m if m >= 0 else np.zeros(T, bool))
    steps = lambda seg: sum((int(rank[a]) + 31) // 32 for a in set(tok[seg].tolist()) if a >= 0)
    def cost(order):
        per = [steps(order[i:i + 64]) for i in range(0, T, 64)]
        return sum(max(per[i:i + 4]) for i in range(0, len(per), 4)), max(per)
    by_adapter = np.concatenate([v["perm"], np.nonzero((tok < 0) & carries)[0], np.nonzero((tok < 0) & ~carries)[0]])
    assert all(g <= s for g, s in zip(cost(order), cost(by_adapter)))
    if len(lengths) > 40:
        assert cost(order)[0] < cost(by_adapter)[0]      # (what it is for)
    for i in range(0, T, 64):
        a = tok[order[i:i + 64]]
        assert len(set(a.tolist())) == 1 + int(np.sum(a[1:] != a[:-1]))
    # rows without a delta fill whole blocks of 256, but for one block that has both kinds (those without last) and the end
    plain = [~carries[order[i:i + 256]] for i in range(0, T, 256)]
    assert sum(bool(p.any() and not p.all()) for p in plain) <= 1 and all(np.all(np.diff(p.astype(int)) >= 0) for p in plain)


@pytest.mark.parametrize("T,n_a,ranks,K,N,zipf,m,dealt", [
    (5072, 118, (64, 8, 128, 16, 32), 8, 2992, 0.0, -1, False), (10764, 203, (64, 8, 128, 16, 32), 48, 1400, 0.0, -1, False),
    (3286, 65, (16, 32, 64, 128), 64, 4800, 0.0, -1, False), (2559, 77, (64,), 40, 7256, 0.0, 0, False),
    (2623, 120, (16, 32, 64, 128), 64, 5176, 1.1, -1, True), (1812, 122, (16, 32, 64, 128), 16, 6840, 1.1, 0, True)])
def test_rows_of_the_product_by_stage_lists_are_dealt_where_that_is_less(T, n_a, ranks, K, N, zipf, m, dealt):
    """K <= 128 and 192 tiles of 256 x 256 and more: the kernel that walks the stage lists, whose tiles take as long as all their
    adapters' stages.  Single tokens; dealt rows neither raise the longest tile nor take more rounds."""
    assert B.lora_gemm_choice(T, K, N, B.LORA_BF16, True)[0] == 4 and (-(-T // 256)) * (-(-N // 256)) >= 192
    rng = np.random.default_rng(7)
    share = 1.0 / np.arange(1, n_a + 1) ** zipf
    ads = rng.choice(n_a, size=T, p=share / share.sum()).astype(np.int32)
    rank = np.asarray([ranks[a % len(ranks)] for a in range(n_a)], np.int32)
    p = B.lora_plan(T, np.arange(T + 1), ads, rank, np.ones(n_a), K, N, B.LORA_BF16, merged_adapter=m if m >= 0 else None)
    v = B.lora_plan_export(p)
    p.destroy()
    tok, order = v["token_adapter"], v["gemm_order"]
    per_tile = np.diff(v["gemm_stage_offset"])
    carries = (tok >= 0) | (ads != m if m >= 0 else np.zeros(T, bool))
    by_adapter = np.concatenate([v["perm"], np.nonzero((tok < 0) & carries)[0], np.nonzero((tok < 0) & ~carries)[0]])
    def stages(rows):
        own = sum(-(-2 * int(rank[a]) // 64) for a in set(tok[rows].tolist()) if a >= 0)
        return own + (-(-2 * int(rank[m]) // 64) if m >= 0 and carries[rows].any() else 0)
    in_order = np.asarray([stages(by_adapter[i:i + 256]) for i in range(0, T, 256)])
    assert np.array_equal(per_tile, [stages(order[i:i + 256]) for i in range(0, T, 256)])
    if dealt:
        assert per_tile.max() < 0.7 * in_order.max()
    else:
        assert sorted(per_tile) == sorted(in_order)


@pytest.mark.parametrize("T,n_a,r,K", [(300, 3, 64, 11008), (128, 1, 128, 4096), (1100, 4, 16, 4096)])
def test_given_tunables_of_the_streaming_shrink_are_what_it_runs_with(T, n_a, r, K):
    """Batches of few streaming tiles: the number of K parts that shrink_stream_wgs asks for, whether it comes from the
    descriptor, the process defaults or the shape table; without it, the planner's choice."""
    w = wl.random_case(31 + T, T, 8, 512, n_a, (r,), max_seg=T // n_a, frac_none=0.0)
    def plan(**tuning):
        p = B.lora_plan(w.T, w.seg_indptr, w.seg_adapter, w.adapter_rank, w.adapter_scale, K, w.N, B.LORA_BF16, tuning=tuning)
        v = B.lora_plan_export(p)
        assert B.lora_plan_query(p)[1] == v["v_parts"] * T * v["v_row_stride"] * 4
        p.destroy()
        return v
    def tiles(wgs):                                          # 64-token tiles where 128-token tiles are fewer than wgs / 4
        groups = np.diff(v["group_offset"])
        return int(np.sum(-(-groups // (64 if 4 * np.sum(-(-groups // 128)) < wgs else 128))))
    v = plan()
    for wgs in (2, 40, 100, 511, 4000):
        want = 1
        while want < 4 and tiles(wgs) * want < max(1, wgs // 2) and K // 32 // (2 * want) >= 8:
            want *= 2
        assert plan(shrink_stream_wgs=wgs)["v_parts"] == want, wgs
        default = B.lora_tuning_get()["shrink_stream_wgs"]
        B.lora_tuning_set(shrink_stream_wgs=wgs)
        try:
            assert plan()["v_parts"] == want, wgs
        finally:
            B.lora_tuning_set(shrink_stream_wgs=default)
        B.lora_tuning_table_set([dict(tokens=T, k=K, n=w.N, max_rank=r, group_class=gc, tunables=dict(shrink_stream_wgs=wgs)) for gc in (0, 1, 2)])
        try:
            assert plan()["v_parts"] == want, wgs
        finally:
            B.lora_tuning_table_set(None)
    assert plan()["v_parts"] == v["v_parts"]


@pytest.mark.parametrize("name", ["cfg1", "cfg2", "cfg3", "cfg4", "cfg4d", "cfg5"])
def test_config_tables_bit_exact(name):
    w = wl.CONFIGS[name](with_w=False) if name != "cfg5" else wl.cfg5("attn", with_w=False)
    # matrices are not needed here; the tables only depend on the integer structure
    v, q = _export(w)
    tok, perm = _check_tables(w, v)
    _check_tiles(w, v, tok, perm)
    _check_gemm_tables(w, v, tok, perm)
    R = max(8, (int(w.adapter_rank.max()) + 7) // 8 * 8)
    assert q[0] == R and q[1] == v["v_parts"] * w.T * R * 4 and q[2] >= q[1] and q[2] % 256 == 0
    expect = B.LORA_VARIANT_GENERAL if w.dtype == "f32" else B.LORA_VARIANT_TILED
    assert v["kernel_family"] == expect


@settings(max_examples=150, deadline=None)
@given(st.lists(st.tuples(st.integers(0, 40), st.integers(-1, 5)), min_size=0, max_size=20),
       st.lists(st.sampled_from([0, 8, 16, 24, 32, 64, 128]), min_size=6, max_size=6) |
       st.lists(st.sampled_from([0, 3, 8, 20, 100, 129, 256]), min_size=6, max_size=6),     # also ranks only the shrink tiles
       st.sampled_from([64, 200, 1000]))
def test_random_tables_and_tiles(segs, ranks, N):
    lengths = [s[0] for s in segs]
    ads = [s[1] for s in segs]
    T = sum(lengths)
    indptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32) if segs else np.zeros(1, np.int32)
    w = wl.Workload("h", "bf16", T, 64, N, indptr, np.asarray(ads, np.int32), np.asarray(ranks, np.int32),
                    np.ones(6, np.float32), np.zeros((T, 64), np.float32), None)
    v, _ = _export(w, B.LORA_VARIANT_TILED)
    tok, perm = _check_tables(w, v)
    _check_tiles(w, v, tok, perm)
    _check_gemm_tables(w, v, tok, perm)


def test_plan_is_deterministic():
    w = wl.cfg4(with_w=False)
    a, _ = _export(w)
    b, _ = _export(w)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


def test_unaligned_layouts_take_general_kernels():
    base = dict(seed=1, T=10, N=32, n_a=2, with_w=False)
    G, T_ = B.LORA_VARIANT_GENERAL, B.LORA_VARIANT_TILED
    fam = lambda v: (v["kernel_family"], v["shrink_kernel_family"])
    w = wl.random_case(K=36, ranks=(8,), **base)           # K not a multiple of 8: nothing is tiled
    assert fam(_export(w)[0]) == (G, G)
    # ranks that only the expand cannot take: the shrink alone keeps the MFMA kernels (tiles for it, none for the expand)
    for ranks in ((5,), (256,), (3, 12, 100, 174)):
        w = wl.random_case(K=64, ranks=ranks, **base)
        for variant in (B.LORA_VARIANT_AUTO, T_):
            v = _export(w, variant)[0]
            assert fam(v) == (G, T_) and v["shrink_tiles"].shape[0] > 0 and v["expand_tiles"].shape[0] == 0
            tok, perm = _check_tables(w, v)
            _check_tiles(w, v, tok, perm)
        assert fam(_export(w, G)[0]) == (G, G)
    wf = wl.random_case(K=64, ranks=(5,), dtype="f32", **base)
    assert fam(_export(wf)[0]) == (G, G)                    # fp32: general throughout
    w = wl.random_case(K=64, ranks=(8,), **base)
    assert fam(_export(w, G)[0]) == (G, G)
    assert fam(_export(w)[0]) == (T_, T_)


def _desc(T=4, indptr=(0, 2, 4), seg_ad=(0, 1), ranks=(8, 16), scales=(1.0, 2.0), k=64, n=64,
          dtype=B.LORA_BF16, variant=0, keep=None):
    keep = keep if keep is not None else []
    i = np.asarray(indptr, np.int32); a = np.asarray(seg_ad, np.int32)
    r = np.asarray(ranks, np.int32); s = np.asarray(scales, np.float32)
    keep.extend([i, a, r, s])
    P = ctypes.POINTER(ctypes.c_int32); F = ctypes.POINTER(ctypes.c_float)
    return B.BatchDesc(T, len(seg_ad), i.ctypes.data_as(P), a.ctypes.data_as(P), len(ranks),
                       r.ctypes.data_as(P), s.ctypes.data_as(F), k, n, dtype, variant), keep


def test_error_paths():
    ok, keep = _desc()
    st_, h = B.lora_plan_create_raw(ok)
    assert st_ == B.LORA_OK and h
    B._lib.lora_plan_destroy(h)
    bad = [
        _desc(indptr=(1, 2, 4)),            # does not start at 0
        _desc(indptr=(0, 3, 2)),            # decreasing / wrong end
        _desc(indptr=(0, 2, 3)),            # does not end at T
        _desc(seg_ad=(0, 2)),               # adapter id out of range
        _desc(seg_ad=(0, -2)),
        _desc(ranks=(8, 257)),              # rank beyond LORA_MAX_RANK
        _desc(ranks=(8, -1)),
        _desc(scales=(1.0, float("nan"))),
        _desc(scales=(float("inf"), 1.0)),
        _desc(k=0), _desc(n=0), _desc(dtype=7), _desc(variant=9), _desc(T=-1),
    ]
    for d, keep in bad:
        st_, h = B.lora_plan_create_raw(d)
        assert st_ == B.LORA_ERR_INVALID_ARG and not h
    assert B.lora_plan_create_raw(None)[0] == B.LORA_ERR_INVALID_ARG
    for bad_m in (3, -1):                            # two adapters: 0 (none), 1 and 2 are the valid values
        d, keep = _desc()
        d.merged_adapter_plus1 = bad_m
        assert B.lora_plan_create_raw(d)[0] == B.LORA_ERR_INVALID_ARG
    d, keep = _desc()
    d.seg_indptr = None
    assert B.lora_plan_create_raw(d)[0] == B.LORA_ERR_INVALID_ARG
    assert B._lib.lora_plan_query(None, None, None, None) == B.LORA_ERR_INVALID_ARG
    B._lib.lora_plan_destroy(None)           # allowed
    assert B.lora_status_str(B.LORA_ERR_WORKSPACE).startswith("workspace")
    # empty batch and empty segments are valid
    st_, h = B.lora_plan_create_raw(_desc(T=0, indptr=(0,), seg_ad=())[0])
    assert st_ == B.LORA_OK
    B._lib.lora_plan_destroy(h)
    st_, h = B.lora_plan_create_raw(_desc(T=4, indptr=(0, 0, 4, 4), seg_ad=(0, 1, 0))[0])
    assert st_ == B.LORA_OK
    B._lib.lora_plan_destroy(h)


def test_compute_calls_reject_bad_arguments_without_a_gpu():
    w = wl.random_case(2, 12, 64, 64, 2, (8,), with_w=False)
    p = device.make_plan(w)
    L = B._lib
    assert L.lora_shrink(p.handle, None, 64, None, None, None) == B.LORA_ERR_INVALID_ARG
    assert L.lora_shrink(None, 256, 64, 256, 256, None) == B.LORA_ERR_INVALID_ARG
    assert L.lora_shrink(p.handle, 256, 32, 256, 256, None) == B.LORA_ERR_INVALID_ARG       # ldx < K
    assert L.lora_expand(p.handle, 256, 256, 256, 64, ctypes.c_float(0.5), None) == B.LORA_ERR_INVALID_ARG   # beta
    assert L.lora_expand(p.handle, 256, 256, 256, 32, ctypes.c_float(1.0), None) == B.LORA_ERR_INVALID_ARG   # ldy < N
    assert L.lora_base_gemm(4, 0, 4, B.LORA_BF16, 256, 8, 256, 8, 256, 8, None) == B.LORA_ERR_INVALID_ARG
    assert L.lora_fused_forward(p.handle, 256, 64, 256, 64, 256, 256, 256, 64, 256, 16, None) == B.LORA_ERR_WORKSPACE
    p.destroy()
    # lora_merge(L, n, k, rank, scale, dtype, variant, Wt_ptrs, ldw, At_ptrs, Bt_ptrs, stream)
    f = ctypes.c_float
    assert L.lora_merge(2, 64, 64, 8, f(1.0), B.LORA_BF16, B.LORA_VARIANT_AUTO, None, 64, 256, 256, None) == B.LORA_ERR_INVALID_ARG
    assert L.lora_merge(2, 64, 64, 8, f(1.0), B.LORA_BF16, B.LORA_VARIANT_AUTO, 256, 32, 256, 256, None) == B.LORA_ERR_INVALID_ARG   # ldw < k
    assert L.lora_merge(2, 64, 64, 8, f(float("nan")), B.LORA_BF16, B.LORA_VARIANT_AUTO, 256, 64, 256, 256, None) == B.LORA_ERR_INVALID_ARG
    assert L.lora_merge(2, 64, 64, 300, f(1.0), B.LORA_BF16, B.LORA_VARIANT_AUTO, 256, 64, 256, 256, None) == B.LORA_ERR_INVALID_ARG  # rank
    assert L.lora_merge(2, 64, 60, 8, f(1.0), B.LORA_BF16, B.LORA_VARIANT_TILED, 256, 64, 256, 256, None) == B.LORA_ERR_UNSUPPORTED   # k % 8
    assert L.lora_merge(2, 64, 64, 8, f(1.0), B.LORA_F32, B.LORA_VARIANT_TILED, 256, 64, 256, 256, None) == B.LORA_ERR_UNSUPPORTED
    assert L.lora_merge(0, 64, 64, 8, f(1.0), B.LORA_BF16, B.LORA_VARIANT_AUTO, None, 64, None, None, None) == B.LORA_OK             # no layers
    assert L.lora_merge(2, 64, 64, 0, f(1.0), B.LORA_BF16, B.LORA_VARIANT_AUTO, None, 64, None, None, None) == B.LORA_OK             # rank 0


def test_mixture_delta_is_refused_before_any_launch():
    """A lora_delta whose two shrinks go in one launch: every bad argument of the second step is seen before the first one
    runs.  (Without a GPU a call that gets as far as its plan's upload returns LORA_ERR_DEVICE.)"""
    w = wl.random_case(3, 1200, 1024, 256, 4, (16, 64), max_seg=200, with_w=False)
    p = device.make_plan(w, merged_adapter=0)
    v = B.lora_plan_export(p)
    for tiles in (v["shrink_tiles"], v["unmerge_shrink_tiles"]):       # (only the streaming shrink's tiles hold more than 32 tokens)
        assert len(tiles) and tiles[:, 2].max() > 32
    good = dict(x=4096, At=1 << 24, Bt=1 << 25, v=1 << 26, y=1 << 30, ldy=256)
    for bad in (dict(Bt=None), dict(At=None), dict(y=None), dict(v=None), dict(ldy=255), dict(y=(1 << 30) + 1), dict(Bt=(1 << 25) + 4), dict(v=(1 << 26) + 4)):
        a = dict(good, **bad)
        st = B._lib.lora_delta(p.handle, a["x"], 1024, a["At"], a["Bt"], a["v"], a["y"], a["ldy"], ctypes.c_float(1.0), None)
        assert st == B.LORA_ERR_INVALID_ARG, bad
    p.destroy()


def test_tuning_roundtrip_changes_tiles():
    before = B.lora_tuning_get()
    try:
        B.lora_tuning_table_set([dict(tokens=0, k=1, n=1, max_rank=8, group_class=0, tunables={})])   # no entry applies
        w = wl.cfg3(with_w=False)
        a = _export(w)[0]
        B.lora_tuning_set(shrink_tb2_min_rows=1 << 20, shrink_tb4_min_rows=1 << 20, expand_tb2_min_rows=1 << 20,
                          shrink_small_waves=4, shrink_target_wgs=1,
                          shrink_small_jb=2, shrink_stream_min_tokens=1 << 30)
        b = _export(w)[0]
        assert b["shrink_waves"] == 4
        assert b["shrink_tiles"].shape[0] // b["v_parts"] > a["shrink_tiles"].shape[0] // a["v_parts"]
        assert b["expand_tiles"].shape[0] > a["expand_tiles"].shape[0]
        tok, perm = _check_tables(w, b)
        _check_tiles(w, b, tok, perm)
    finally:
        B.lora_tuning_set(**before)
        B.lora_tuning_table_set([])
    assert B.lora_tuning_get() == before


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "lora_abi.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    names = set(re.findall(r"\b(lora_[a-z_]+)\s*\(", hdr))
    assert {"lora_plan_create", "lora_shrink", "lora_expand", "lora_fused_forward"} <= names
    for n in sorted(names):
        assert hasattr(B._lib, n), f"{n} is declared in lora_abi.h but not exported"
    assert names == set(B.EXPORTED)


def test_trace_set_checks_its_arguments_without_a_gpu():
    import ctypes
    buf = (ctypes.c_int64 * 16)()
    base = ctypes.addressof(buf)
    assert B._lib.lora_trace_set(ctypes.c_void_p(base + 4), 64) == B.LORA_ERR_INVALID_ARG      # not 8-byte aligned
    assert B._lib.lora_trace_set(ctypes.c_void_p(base), 0) == B.LORA_ERR_INVALID_ARG           # no room at all
    assert B._lib.lora_trace_set(None, 0) == B.LORA_OK                                         # off (the default)


def test_shape_table_is_consulted_inside_plan_create():
    """The shape-keyed table (paper section 4.3.2): lora_plan_create looks the batch's class up -- tokens with an
    adapter (smallest entry at or above, else the largest), K, N, rank class, group class -- and plans with the
    entry on top of the process defaults; values in the descriptor override both; every plan keeps its snapshot."""
    defaults = B.lora_tuning_get()
    shipped = B.lora_tuning_table_get()
    assert all(set(e["tunables"]) <= set(B.TUNING_FIELDS) for e in shipped)
    w = wl.cfg2(with_w=False)                                   # 256 tokens, 4096 -> 4096, ranks up to 64, decode-shaped
    try:
        B.lora_tuning_table_set([
            dict(tokens=128, k=4096, n=4096, max_rank=64, group_class=0, tunables={"expand_wave_bytes": 4096}),
            dict(tokens=512, k=4096, n=4096, max_rank=64, group_class=0, tunables={"expand_wave_bytes": 32768, "fused_delay": 7}),
            dict(tokens=1024, k=4096, n=4096, max_rank=64, group_class=0, tunables={"expand_wave_bytes": 65536}),
            dict(tokens=512, k=4096, n=4096, max_rank=64, group_class=1, tunables={"expand_wave_bytes": 8192}),
            dict(tokens=512, k=4096, n=4096, max_rank=32, group_class=0, tunables={"expand_wave_bytes": 8192}),
            dict(tokens=512, k=4096, n=11008, max_rank=64, group_class=0, tunables={"expand_wave_bytes": 8192}),
        ])
        assert len(B.lora_tuning_table_get()) == 6
        p = device.make_plan(w)
        v = B.lora_plan_export(p)
        assert v["tuning_source"] == 1
        assert v["tuning"]["expand_wave_bytes"] == 32768 and v["tuning"]["fused_delay"] == 7      # the 512-token entry
        assert v["tuning"]["shrink_target_wgs"] == defaults["shrink_target_wgs"]                   # not in the entry
        n_tab = v["expand_tiles"].shape[0]
        # the descriptor's own values win over the entry
        q = device.make_plan(w, tuning={"expand_wave_bytes": 8192})
        vq = B.lora_plan_export(q)
        assert vq["tuning_source"] == 3 and vq["tuning"]["expand_wave_bytes"] == 8192 and vq["tuning"]["fused_delay"] == 7
        assert vq["expand_tiles"].shape[0] > n_tab                                                 # smaller tiles, more of them
        tok, perm = _check_tables(w, vq)
        _check_tiles(w, vq, tok, perm)
        # beyond the largest bucket: the largest entry; a shape class without entry: defaults
        big = wl.random_case(5, 1500, 4096, 4096, 600, (8, 64), max_seg=1, with_w=False)
        assert B.lora_plan_export(device.make_plan(big))["tuning"]["expand_wave_bytes"] == 65536
        other = wl.random_case(6, 100, 512, 512, 30, (8, 64), max_seg=1, with_w=False)
        vo = B.lora_plan_export(device.make_plan(other))
        assert vo["tuning_source"] == 0 and vo["tuning"] == defaults
        # group classes: 0 every adapter group below 64 tokens, 2 groups of 512 tokens or more on average, 1 between;
        # an entry without values is a match that keeps the defaults (and is not reported as a source)
        B.lora_tuning_table_set([
            dict(tokens=4096, k=4096, n=4096, max_rank=64, group_class=1, tunables={"expand_stream_stages": 8}),
            dict(tokens=4096, k=4096, n=4096, max_rank=64, group_class=2, tunables={"expand_stream_stages": 32}),
            dict(tokens=2048, k=4096, n=4096, max_rank=64, group_class=2, tunables={}),
        ])
        long_requests = wl.cfg3(with_w=False)                                       # 4 adapters x 1024 tokens
        assert B.lora_plan_export(device.make_plan(long_requests))["tuning"]["expand_stream_stages"] == 32
        mixed = wl.random_case(7, 4096, 4096, 4096, 40, (64,), max_seg=200, with_w=False)   # about 100 tokens per adapter
        assert B.lora_plan_export(device.make_plan(mixed))["tuning"]["expand_stream_stages"] == 8
        half = wl.random_case(8, 2048, 4096, 4096, 2, (64,), max_seg=2048, with_w=False)
        half = wl.Workload("h", "bf16", 2048, 4096, 4096, np.array([0, 1024, 2048], np.int32), np.array([0, 1], np.int32),
                           half.adapter_rank, half.adapter_scale, half.x, None)
        vh = B.lora_plan_export(device.make_plan(half))
        assert vh["tuning_source"] == 0 and vh["tuning"] == defaults                 # the row of zeros, not the 4096-token entry
        # replacing the table does not touch plans already made
        B.lora_tuning_table_set([])
        assert B.lora_plan_export(p)["tuning"]["expand_wave_bytes"] == 32768
        assert B.lora_tuning_table_get() == shipped
        with pytest.raises(B.LoraError):
            B.lora_tuning_table_set([dict(tokens=64, k=64, n=64, max_rank=48, group_class=0, tunables={})])   # not a rank class
        with pytest.raises(KeyError):
            B.lora_tuning_table_set([dict(tokens=64, k=64, n=64, max_rank=64, group_class=0, tunables={"no_such_tunable": 1})])
    finally:
        B.lora_tuning_table_set([])
    assert B.lora_tuning_get() == defaults


def test_build_refuses_scratch_in_kernels_that_count_their_loads():
    """build.py's guard: a kernel that waits with hand-written s_waitcnt vmcnt(n) must not spill (scratch accesses
    use the same counter); the compiler's resource report is parsed and a nonzero scratch size fails the build."""
    from paper_2411_00915_amd import build as b
    R = b.REMARK
    head = f"k.hip:1:1: remark: Function Name: _ZN12_GLOBAL__N_116gemm_ring_kernelILb1EEEv {R}"
    other = f"k.hip:9:1: remark: Function Name: _ZN12_GLOBAL__N_117gemm_tiled_kernelILi4ELb0ELb0EEEv {R}"
    ok = [head, f"k.hip:1:1: remark:     ScratchSize [bytes/lane]: 0 {R}", f"k.hip:1:1: remark:     VGPRs Spill: 0 {R}",
          other, f"k.hip:9:1: remark:     ScratchSize [bytes/lane]: 64 {R}"]
    b._check_no_scratch("k.hip", ok, ("gemm_ring_kernel",))          # other kernels may use scratch
    for bad in ("ScratchSize [bytes/lane]: 8", "VGPRs Spill: 3"):
        with pytest.raises(RuntimeError):
            b._check_no_scratch("k.hip", [head, f"k.hip:1:1: remark:     {bad} {R}"], ("gemm_ring_kernel",))
    with pytest.raises(RuntimeError):                                  # no report at all: cannot vouch for it
        b._check_no_scratch("k.hip", [other], ("gemm_ring_kernel",))
    assert b._without_remarks(ok + ["  459 | {", "      | ^", "2 remarks generated when compiling for gfx950.", "real warning"]) == ["real warning"]


def test_streaming_tiles_for_small_batches_with_long_groups():
    """Below shrink_stream_min_tokens the planner still picks the streaming tiles (up to 128 tokens of one adapter
    over all its rank rows) when the batch cannot run as the single decode launch and holds a group of 64 tokens
    or 128 tokens in all; batches of short groups keep the 16-token tiles; 2^30 switches streaming off."""
    def shrink_rows(T, n_a, r, **tune):
        before = B.lora_tuning_get()
        try:
            if tune:
                B.lora_tuning_set(**tune)
            seg = np.linspace(0, T, n_a + 1).astype(np.int32)
            w = wl.Workload("s", "bf16", T, 4096, 4096, seg, np.arange(n_a, dtype=np.int32), np.full(n_a, r, np.int32),
                            np.ones(n_a, np.float32), np.zeros((T, 4096), np.float32), None)
            v, _ = _export(w, B.LORA_VARIANT_TILED)
            tok, perm = _check_tables(w, v)
            _check_tiles(w, v, tok, perm)
            return int(v["shrink_tiles"][:, 2].max()), int(v["shrink_tiles"][:, 4].max())     # tokens, rank rows of the largest tile
        finally:
            B.lora_tuning_set(**before)
    # (a streaming tile spans all rank rows of its adapter; the other family's tiles at most 64)
    assert shrink_rows(256, 1, 128) == (64, 128)                # one group of 256 tokens: streaming, 64-token tiles (few workgroups)
    assert shrink_rows(64, 1, 128) == (64, 128)                 # one group of 64 tokens
    assert shrink_rows(256, 16, 128) == (16, 128)               # 16 tokens per group, rank 128, 256 tokens in all: streaming
    assert shrink_rows(256, 16, 64)[0] == 16 and shrink_rows(256, 16, 64)[1] <= 32   # short groups, ranks <= 64: 16-token tiles of the decode launch
    assert shrink_rows(48, 4, 128)[1] <= 64                     # 48 tokens in groups of 12: too small for the streaming kernels
    assert shrink_rows(256, 1, 128, shrink_stream_min_tokens=1 << 30)[1] <= 64       # streaming switched off


def test_small_gemm_shapes_cover_every_tile():
    """The shapes of the GPU tests of the GEMM that splits K over its wavefronts pick every tile it has: in bf16 with
    ranks of the tuned kernels (even token counts) and with others (odd ones), and in fp32."""
    from test_gpu_parity import SMALL_GEMM_SHAPES
    tiles = {(4, 4), (2, 4), (4, 2), (2, 2), (4, 1), (1, 2), (1, 1)}
    for odd in (0, 1):
        picked = [B.lora_gemm_choice(T, K, N, B.LORA_BF16, True) for T, K, N in SMALL_GEMM_SHAPES if T % 2 == odd]
        assert {c[1:] for c in picked if c[0] == 1} == tiles, odd
    assert {B.lora_gemm_choice(T, K, N, B.LORA_F32, True)[1:] for T, K, N in SMALL_GEMM_SHAPES if K >= 32} == tiles


def _layer_batch(T, K, N, n_a, ranks, max_seg, **kw):
    w = wl.random_case(77 + T + n_a, T, K, N, n_a, ranks, max_seg=max_seg, with_w=False)
    return w, device.make_plan(w, **kw)


@pytest.mark.parametrize("T,K,N,n_a,ranks,max_seg,tile,own", [
    (64, 1032, 4096, 1, (128,), 64, (2, 2), False), (250, 1096, 4096, 5, (8, 16, 128), 150, (4, 4), False),
    (300, 4096, 4096, 2, (64,), 300, (4, 4), False), (37, 584, 4096, 9, (8, 16, 40, 64), 5, (2, 2), True),
    (1, 4096, 4096, 1, (64,), 1, (1, 1), True), (200, 264, 4104, 40, (8, 64), 5, (4, 2), True)])
def test_layer_shrink_tiles_cover_the_batch_once(T, K, N, n_a, ranks, max_seg, tile, own):
    """The tiles that go into the product's launch: 16 tokens x up to 32 rank rows, every (token, rank row) in one of them."""
    assert B.lora_gemm_choice(T, K, N, B.LORA_BF16, True) == (1, *tile)
    w, p = _layer_batch(T, K, N, n_a, ranks, max_seg)
    v, tiles, extra = B.lora_plan_export(p), B.lora_layer_shrink_tiles(p, own=True), B.lora_layer_shrink_tiles(p)
    p.destroy()
    tok, perm = _check_tables(w, v)
    assert len(tiles) and len(extra) == (0 if own else len(tiles))
    for part in range(v["v_parts"] if own else 1):
        mine = [tuple(t[:5]) for t in tiles if not own or (t[5] >> 8) & 15 == part]
        plan_ref.check_cover(mine, tok, perm, int(w.adapter_rank.max()), adapter_rank=w.adapter_rank, rank_axis=True)
    for t in tiles:
        tb, jb = t[5] & 15, (t[5] >> 4) & 15
        assert tb == 1 and t[2] <= 16 and jb in (1, 2) and t[4] <= 16 * jb and t[3] % 16 == 0
        assert t[6] == w.adapter_rank[t[0]] and np.int32(t[7]).view(np.float32) == w.adapter_scale[t[0]]


@pytest.mark.parametrize("T,K,N,n_a,ranks,max_seg,merged", [
    (100, 4096, 4096, 5, (104, 128), 50, None),          # the product's tile is the one that keeps two launches
    (512, 4096, 11008, 5, (64, 128), 200, None),         # another GEMM's product
    (177, 2040, 1264, 128, (128,), 1, None),             # the shrink would crowd the product
    (600, 2048, 2048, 3, (64, 128), 300, None),          # more than 512 tokens
    (37, 584, 4096, 9, (8, 16, 40, 64), 5, 1),           # mixture mode: neither the own branches nor the removal
    (200, 4096, 4096, 3, (64, 128), 90, 0)])
def test_layer_shrink_tiles_are_built_only_where_they_are_read(T, K, N, n_a, ranks, max_seg, merged):
    w, p = _layer_batch(T, K, N, n_a, ranks, max_seg, merged_adapter=merged)
    v = B.lora_plan_export(p)
    assert v["kernel_family"] == B.LORA_VARIANT_TILED
    if merged is None:                                                    # not of that size themselves
        assert v["shrink_tiles"][:, 2].max() > 16 or v["shrink_tiles"][:, 4].max() > 32
    else:
        assert v["num_unmerge"] > 0
    for removal in (False, True):
        assert len(B.lora_layer_shrink_tiles(p, removal)) == 0 and len(B.lora_layer_shrink_tiles(p, removal, own=True)) == 0
    p.destroy()


@pytest.mark.parametrize("T,n_a,ranks,N,rows,blocks", [
    # up to rank 32: 16 tokens, one, two and four blocks of 256 features
    (700, 2, (30, 4), 4096, 16, 1), (1100, 2, (31, 12), 4096, 16, 2), (2800, 2, (27, 20), 4096, 16, 4), (1500, 200, (31,), 11008, 16, 4),
    # odd ranks above 24: 32 tokens where tiles of 16 are 1024 and fewer or tiles of 32 are 3072 and more
    (700, 2, (31, 9), 4096, 32, 1), (1018, 1, (31,), 4096, 32, 1), (260, 1, (25,), 13824, 32, 1), (4800, 2, (25,), 11008, 32, 6), (2400, 1, (31,), 11008, 32, 3),
    # higher ranks of about one length: a full round of two or four blocks, for requests of eight tokens a tile on average
    (1500, 2, (100,), 4096, 32, 2), (3600, 3, (200, 256), 4096, 32, 4), (270, 108, (100,), 4096, 32, 1), (280, 90, (200, 256), 5120, 32, 1),
    (380, 60, (200, 256), 3712, 32, 1), (900, 60, (200, 256), 3712, 32, 2),
    # two blocks up to 768 tiles of them, odd ranks up to 512, else four up to 512 of them
    (3040, 1, (160,), 4096, 32, 2), (2000, 1, (100,), 4096, 32, 2), (2200, 1, (101,), 4096, 32, 1), (1130, 1, (256,), 11008, 32, 4), (3300, 1, (101,), 4096, 32, 4)])
def test_tiles_of_the_expand_for_rows_of_any_length(T, n_a, ranks, N, rows, blocks):
    """Tokens and features of the largest tile, and that the tiles are every row and feature of every adapter once."""
    lengths = np.full(n_a, T // n_a)
    lengths[:T % n_a] += 1
    rank = np.asarray([ranks[a % len(ranks)] for a in range(n_a)], np.int32)
    p = B.lora_plan(T, np.concatenate([[0], np.cumsum(lengths)]), np.arange(n_a), rank, np.ones(n_a), 512, N, B.LORA_BF16)
    fn, ptr = B._lib.lora_rows_expand_tiles, ctypes.POINTER(B.Tile)()
    fn.argtypes, fn.restype = [ctypes.c_void_p, ctypes.c_void_p], ctypes.c_int32
    tiles = [ptr[i] for i in range(fn(p.handle, ctypes.byref(ptr)))]
    group = dict(zip(range(n_a), zip(np.cumsum(lengths) - lengths, np.cumsum(lengths))))
    covered = np.zeros((T, -(-N // 256)), np.int32)
    for t in tiles:
        lo, hi = group[t.adapter]
        assert lo <= t.row0 and t.row0 + t.nrows <= hi and t.c0 % 256 == 0 and (t.cn % 256 == 0 or t.c0 + t.cn == N)
        covered[t.row0:t.row0 + t.nrows, t.c0 // 256:-(-(t.c0 + t.cn) // 256)] += 1
    assert np.all(covered == 1)
    steps = {t.row0 - group[t.adapter][0] for t in tiles} - {0}
    assert not steps or min(steps) == rows
    if max(lengths) > 16:
        assert max(t.nrows for t in tiles) == min(rows, max(lengths))
    assert max(-(-t.cn // 256) for t in tiles) == min(blocks, -(-N // 256))
    p.destroy()


@pytest.mark.parametrize("lengths,ranks,N,rows_of_long", [
    ((190, 180, 200, 180), (4, 100, 12, 256), 4096, 16), ((40, 33, 30, 17, 16, 1), (4, 100, 12, 256, 20, 129), 13824, 16),
    ((500, 500), (8, 160), 13824, 32), ((300, 300), (256, 200), 8192, 32), ((300, 300), (127, 40), 8192, 32)])
def test_long_ranks_among_short_ones_have_tiles_of_16_tokens_where_that_ends_earlier(lengths, ranks, N, rows_of_long):
    """... of the expand for rows of any length: not where the chip holds no more of them, not where all ranks are long; every
    row and feature of every adapter once."""
    T, n_a = sum(lengths), len(lengths)
    p = B.lora_plan(T, np.concatenate([[0], np.cumsum(lengths)]), np.arange(n_a), np.asarray(ranks, np.int32), np.ones(n_a), 512, N, B.LORA_BF16)
    fn, ptr = B._lib.lora_rows_expand_tiles, ctypes.POINTER(B.Tile)()
    fn.argtypes, fn.restype = [ctypes.c_void_p, ctypes.c_void_p], ctypes.c_int32
    tiles = [ptr[i] for i in range(fn(p.handle, ctypes.byref(ptr)))]
    ends = np.cumsum(lengths)
    covered = np.zeros((T, -(-N // 256)), np.int32)
    for t in tiles:
        lo, hi = ends[t.adapter] - lengths[t.adapter], ends[t.adapter]
        rows = rows_of_long if ranks[t.adapter] > 128 else 32
        assert lo <= t.row0 and (t.row0 - lo) % rows == 0 and t.nrows == min(rows, hi - t.row0)
        covered[t.row0:t.row0 + t.nrows, t.c0 // 256:-(-(t.c0 + t.cn) // 256)] += 1
    assert tiles and np.all(covered == 1)
    p.destroy()


@pytest.mark.parametrize("T,N,ranks,max_seg", [(300, 4104, (16, 64), 150), (1300, 8200, (16, 64, 128), 300), (1500, 9000, (64,), 700),
                                               (8192, 11008, (64, 8, 128, 16, 32), 100), (40000, 1032, (64, 16), 300)])
def test_feature_ranges_of_the_streaming_expand(T, N, ranks, max_seg):
    """Every feature of every token tile once, in equal shares of its stages, the longest tiles first."""
    rng = np.random.default_rng(T + N)
    lengths = []
    while sum(lengths) < T:
        lengths.append(min(T - sum(lengths), int(rng.integers(1, max_seg + 1))))
    rank = np.asarray([ranks[a % len(ranks)] for a in range(24)], np.int32)
    p = B.lora_plan(T, np.concatenate([[0], np.cumsum(lengths)]), rng.integers(0, 24, len(lengths)), rank, np.ones(24), 1024, N, B.LORA_BF16)
    tiles = B.lora_plan_export(p)["expand_tiles"]
    stages, blocks = [], {}
    for adapter, row0, nrows, c0, cn, shape, r, _ in tiles.tolist():
        width = 64 * (shape >> 4 & 15)
        assert c0 % width == 0 and (cn % width == 0 or c0 + cn == N)
        stages.append((3300 + 1130 * -(-cn // width), 4600 + 1360 * -(-cn // width), 5500 + 1330 * -(-cn // width))[0 if r <= 32 else 1 if r <= 64 else 2])
        blocks.setdefault((adapter, row0, nrows, width), []).append((c0, cn))
    assert stages == sorted(stages, reverse=True)
    for (_, _, _, width), ranges in blocks.items():
        ranges.sort()
        assert ranges[0][0] == 0 and ranges[-1][0] + ranges[-1][1] == N
        assert all(a + n == b for (a, n), (b, _) in zip(ranges, ranges[1:])) and len({n for _, n in ranges[:-1]}) <= 1
    p.destroy()


def _launch_end(counts):
    """when 256 compute units are through with the tiles {time: how many}, longest first"""
    free, end = [(0, 256)], 0
    for ns, left in sorted(counts.items(), reverse=True):
        while left:
            at, units = heapq.heappop(free)
            take = min(units, left)
            if take < units:
                heapq.heappush(free, (at, units - take))
            heapq.heappush(free, (at + ns, take))
            left, end = left - take, max(end, at + ns)
    return end


@pytest.mark.parametrize("T,adapters,ranks,N", [
    (1500, 47, (64,), 4096), (6000, 100, (16,), 11008), (8192, 128, (64, 8, 128, 16, 32), 11008), (8192, 257, (64,), 4096),
    (4096, 420, (128,), 13824), (8192, 450, (128,), 11008), (49608, 412, (64,), 11008), (16384, 500, (128,), 11008), (65664, 1, (64,), 11008),
    (71300, 1, (64,), 5120), (66000, 3, (32,), 1032), (20000, 1000, (8, 64), 4096), (40000, 2000, (16, 128), 4096), (3000, 1, (64,), 60000)])
def test_feature_ranges_of_the_streaming_expand_end_the_launch_soon(T, adapters, ranks, N):
    """47 to 2000 token tiles: of all lengths that the ranges could have, none would end the launch more than 2 % sooner, by the
    planner's own times of a tile (3.3, 4.6, 5.5 us and 1.13, 1.36, 1.33 a stage), half of the longest tile for their spread,
    and not before memory is through with y and one reading of Bt at 5 TB/s."""
    lengths = np.full(adapters, T // adapters) + (np.arange(adapters) < T % adapters)
    rank = np.asarray([ranks[a % len(ranks)] for a in range(adapters)], np.int32)
    p = B.lora_plan(T, np.concatenate([[0], np.cumsum(lengths)]), np.arange(adapters), rank, np.ones(adapters), 1024, N, B.LORA_BF16)
    tiles = B.lora_plan_export(p)["expand_tiles"].tolist()
    blocks = {(a, row): (shape >> 4 & 15, r) for a, row, _, _, _, shape, r, _ in tiles}
    p.destroy()
    of_kind = collections.Counter(blocks.values())
    memory = (2 * T + int(rank.sum())) * 2 * N / 5000

    def ns(r, stages):
        return 3300 + 1130 * stages if r <= 32 else 4600 + 1360 * stages if r <= 64 else 5500 + 1330 * stages

    def estimate(counts):
        return max(_launch_end(counts), memory) + max(counts) / 2

    chosen = collections.Counter(ns(r, -(-cn // (64 * (shape >> 4 & 15)))) for _, _, _, _, cn, shape, r, _ in tiles)
    best = None
    for longest in range(1, -(-N // 64) + 1):
        counts = collections.Counter()
        for (chunks, r), n in of_kind.items():
            stages = -(-N // (64 * chunks))
            share = -(-stages // -(-stages // longest))
            counts[ns(r, share)] += n * (stages // share)
            if stages % share:
                counts[ns(r, stages % share)] += n
        best = min(best or 1e18, estimate(counts))
    assert estimate(chosen) <= 1.02 * best, (estimate(chosen), best)


@pytest.mark.parametrize("stages", [1 << 25, 1 << 26, 1 << 29])
@pytest.mark.parametrize("T,adapters,N", [(3000, 1, 4096), (66000, 4, 4096), (1100, 8, 1000)])
def test_given_expand_stages_beyond_any_row(stages, T, adapters, N):
    """Stages whose features are past 32 bits: the tiles of a length that is past every row, too, but small."""
    lengths = np.full(adapters, T // adapters) + (np.arange(adapters) < T % adapters)
    tables = (T, np.concatenate([[0], np.cumsum(lengths)]), np.arange(adapters), np.full(adapters, 64, np.int32), np.ones(adapters), 1024, N, B.LORA_BF16)
    tiles = []
    for given in (stages, 1 << 16):
        p = B.lora_plan(*tables, tuning=dict(expand_stream_stages=given))
        tiles.append(B.lora_plan_export(p)["expand_tiles"])
        p.destroy()
    assert np.array_equal(*tiles) and int(tiles[0][:, 4].min()) > 0


def test_every_length_of_expand_ranges_can_be_given_and_by_rounds_is_a_value_of_its_own():
    """16 stages are a length like 8 and 32 (513 token tiles, so that nothing is halved; the list's end is cut); the default,
    which a descriptor can ask for over another process default, is LORA_EXPAND_BY_ROUNDS; the plan's view says which."""
    tables = (65664, np.array([0, 65664]), np.array([0]), np.full(1, 64, np.int32), np.ones(1), 1024, 11008, B.LORA_BF16)
    before = B.lora_tuning_get()["expand_stream_stages"]
    assert before == B.LORA_EXPAND_BY_ROUNDS

    def ranges(**tuning):
        p = B.lora_plan(*tables, tuning=tuning)
        view = B.lora_plan_export(p)
        p.destroy()
        return view["tuning"]["expand_stream_stages"], view["expand_tiles"]

    for stages in (8, 16, 32):
        told, tiles = ranges(expand_stream_stages=stages)
        assert told == stages and int(tiles[:, 4].max()) == 64 * stages and np.mean(tiles[:, 4] == 64 * stages) > 0.8
    told, tiles = ranges()
    assert told == before and int(tiles[:, 4].max()) % (64 * 16) != 0
    try:
        B.lora_tuning_set(expand_stream_stages=8)
        assert ranges()[0] == 8 and int(ranges()[1][:, 4].max()) == 64 * 8
        again, same = ranges(expand_stream_stages=B.LORA_EXPAND_BY_ROUNDS)
        assert again == before and np.array_equal(same, tiles)
    finally:
        B.lora_tuning_set(expand_stream_stages=before)
    assert np.array_equal(ranges()[1], tiles)


def _expand_launch_end(tiles):
    """of a plan's streaming expand tiles, by the planner's times of a tile, in their order"""
    free, end = [(0, 256)], 0
    for _, _, _, _, cn, shape, r, _ in tiles:
        stages = -(-cn // (64 * (shape >> 4 & 15)))
        at, units = heapq.heappop(free)
        if units > 1:
            heapq.heappush(free, (at, units - 1))
        at += 3300 + 1130 * stages if r <= 32 else 4600 + 1360 * stages if r <= 64 else 5500 + 1330 * stages
        heapq.heappush(free, (at, 1))
        end = max(end, at)
    return end


SEARCHED_EXPAND_RANGES = [(c, v) for *c, v in autotune.read_table(autotune.TABLE_INC) if v[B.TUNING_FIELDS.index("expand_stream_stages")] > 0]


@pytest.mark.parametrize("shape_class,values", SEARCHED_EXPAND_RANGES, ids=lambda p: "-".join(map(str, p)) if len(p) == 5 else "")
def test_shipped_expand_ranges_are_not_far_behind_the_chosen_ones(shape_class, values):
    """An entry of the shipped table that gives the expand's ranges was timed against those that the planner chooses without it;
    by the times of a tile, which know no caches, it may be 10 % behind (entries kept from before the planner chose: up to 49 %)."""
    w = autotune.make_case(*shape_class, seed=4100 + sum(shape_class))
    ends = []
    for tuning in ({}, dict(expand_stream_stages=B.LORA_EXPAND_BY_ROUNDS)):
        p = B.lora_plan(w.T, w.seg_indptr, w.seg_adapter, w.adapter_rank, w.adapter_scale, w.K, w.N, B.LORA_BF16, tuning=tuning)
        view = B.lora_plan_export(p)
        p.destroy()
        assert view["tuning_source"] == (3 if tuning else 1)
        ends.append(_expand_launch_end(view["expand_tiles"].tolist()))
    assert ends[0] <= 1.1 * ends[1], ends


@pytest.mark.parametrize("lengths,ranks,N", [
    ((30, 25, 18, 27, 26, 28), (129, 64), 13824),                    # 324 tiles, 486 with those of rank 129 in 16 tokens: a half more
    ((499, 500), (256, 100), 4096),                                  # 512, 768: as many as have a place, but a half more
    ((60,) + 12 * (30,), (160,) + 12 * (8,), 13824)])                # 756, 864: more than have a place
def test_long_ranks_stay_in_tiles_of_32_tokens_where_these_are_too_many_more(lengths, ranks, N):
    T, n_a = sum(lengths), len(lengths)
    rank = np.asarray([ranks[a % len(ranks)] for a in range(n_a)], np.int32)
    p = B.lora_plan(T, np.concatenate([[0], np.cumsum(lengths)]), np.arange(n_a), rank, np.ones(n_a), 512, N, B.LORA_BF16)
    fn, ptr = B._lib.lora_rows_expand_tiles, ctypes.POINTER(B.Tile)()
    fn.argtypes, fn.restype = [ctypes.c_void_p, ctypes.c_void_p], ctypes.c_int32
    tiles = [ptr[i] for i in range(fn(p.handle, ctypes.byref(ptr)))]
    long_tiles = [t for t in tiles if rank[t.adapter] > 128]
    assert long_tiles and max(t.nrows for t in long_tiles) > 16
    p.destroy()
