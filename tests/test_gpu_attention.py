"""GPU parity: dream_tree_verify_attn and dream_draft_xattn against the float64 oracle on identical
seeded inputs.  Tolerances (max-abs): 1e-5 for float32 tensors, 2e-2 for bf16 tensors."""
import re

import numpy as np
import pytest

import dream_inputs as di
import oracle
from tests.attn_cases import (EXTRA_W8_CASES, FULL_VERIFY_PLANS, FULL_XATTN_PLANS, STREAMING_PLANS, VARIANT_CASES, variant_config,
                              variant_prefix_lens)

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from tests import gpu_util
    return gpu_util


def _cfg(name, dtype, B, Hq, Hkv, D, v, q, T, depth, idx):
    return di.Config(name, dtype, B, Hq, Hkv, D, Hq * D, v, q, T, depth, 1, 4, 1000, 1, idx)


def test_tiny_config_verify_all_elements(gu):
    cfg = di.CONFIGS["tiny"]
    x = di.verify_inputs(cfg)
    got, lse = gu.run_verify(x)
    want, want_lse = oracle.tree_attn(x.q, x.k, x.v, cfg.dtype, x.prefix_len, x.parent, True)
    assert np.abs(got - want).max() <= TOL["f32"]
    assert np.abs(lse - want_lse).max() <= 1e-5


SMALL_CASES = [
    # name, B, Hq, Hkv, D, v, q, T, depth, prefix_len, splits
    ("mha128", 2, 4, 4, 128, 150, 43, 60, 6, [193, 101], 0),
    ("mha128_nosplit", 2, 4, 4, 128, 150, 43, 60, 6, [193, 101], 1),
    ("mha128_3split", 1, 2, 2, 128, 300, 77, 60, 6, [377], 3),
    ("gqa4_128", 2, 8, 2, 128, 130, 31, 60, 6, [161, 64], 0),
    ("gqa2_256", 1, 4, 2, 256, 120, 45, 60, 6, [165], 0),
    ("gqa2_256_nosplit", 2, 4, 2, 256, 70, 13, 33, 5, [83, 40], 1),
    ("mha64", 2, 4, 4, 64, 200, 57, 60, 6, [257, 130], 0),
    ("gqa8_64", 1, 8, 1, 64, 100, 30, 64, 6, [130], 2),
    ("t1", 2, 4, 2, 128, 90, 9, 1, 0, [99, 17], 0),
    ("t17", 1, 4, 2, 128, 90, 9, 17, 4, [99], 2),
    ("paper_tree33", 1, 4, 4, 128, 144, 40, 33, 6, [184], 0),
    ("empty_prefix", 1, 2, 2, 64, 0, 0, 20, 4, [0], 0),
    ("long_mha64", 1, 8, 8, 64, 2900, 140, 60, 6, [3040], 0),        # 97 key tiles, still one launch at head_dim 64
    ("long_gqa4_128", 1, 16, 4, 128, 2500, 60, 60, 6, [2560], 0),    # 82 key tiles, grouped queries
    ("longer_mha128", 1, 8, 8, 128, 2500, 60, 60, 6, [2560], 0),     # past the single-launch limit: key splits and merge
    ("pairs320_mha64", 5, 16, 16, 64, 150, 43, 60, 6, [193, 101, 64, 180, 33], 0),   # more (head, tile) pairs than CUs
    ("pairs288_gqa128", 3, 24, 8, 128, 100, 30, 60, 6, [130, 77, 101], 0),            # 12 query tiles per KV head, in pairs
    ("pairs_odd_tiles", 6, 16, 16, 128, 100, 30, 40, 5, [130, 77, 101, 64, 90, 33], 0),   # 3 query tiles per head: a pair with one tile missing
]


@pytest.mark.parametrize("case", SMALL_CASES, ids=[c[0] for c in SMALL_CASES])
def test_bf16_verify_all_elements(gu, case):
    import paper_2505_19201_amd as dream
    name, B, Hq, Hkv, D, v, q, T, depth, pl, splits = case
    cfg = _cfg(name, "bf16", B, Hq, Hkv, D, v, q, T, depth, 40)
    parents = None
    if name == "paper_tree33":
        parents = di.kary_budget_tree()[None]
    x = di.verify_inputs(cfg, prefix_len=pl, parents=parents)
    dream.dream_set_kv_splits(splits)
    try:
        got, lse = gu.run_verify(x)
    finally:
        dream.dream_set_kv_splits(0)
    want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= TOL["bf16"], np.abs(got - want).max()
    assert np.abs(lse - want_lse).max() <= 2e-3


def test_explicit_tree_mask_matches_parent_derived_mask(gu):
    cfg = _cfg("mask", "bf16", 2, 4, 2, 128, 100, 30, 60, 6, 41)
    x = di.verify_inputs(cfg)
    base, _ = gu.run_verify(x)
    masks = np.stack([di.ancestor_mask_bits(x.parent[b], True)[:, 0] for b in range(cfg.batch)])
    got, _ = gu.run_verify(x, tree_mask=masks)
    assert np.array_equal(got, base)
    # a mask that differs from the tree is honoured: pass the star tree's mask with the original parents
    star = di.star_tree(cfg.n_tree)
    star_mask = np.stack([di.ancestor_mask_bits(star, True)[:, 0]] * cfg.batch)
    got2, _ = gu.run_verify(x, tree_mask=star_mask)
    want, _ = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, np.stack([star] * cfg.batch), True)
    assert np.abs(got2 - want).max() <= TOL["bf16"]
    assert np.abs(got2 - base).max() > 1e-3


def test_trees_above_64_nodes(gu):
    """130-node trees (three mask words in use): the mask derived from `parent`, the same mask given explicitly
    ([B, n_tree, 3] words), a foreign explicit mask, and cross-attention levels whose few query rows name nodes of the
    wide tree; float32 tensors as well."""
    cfg = _cfg("wide130", "bf16", 2, 4, 2, 128, 90, 21, 130, 9, 44)
    x = di.verify_inputs(cfg, prefix_len=[111, 60])
    assert gu.verify_plan(x).startswith("attn_bf16_kernel<128,1,1,2,4,4> ")
    base, lse = gu.run_verify(x)
    want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
    assert np.abs(base - want).max() <= TOL["bf16"] and np.abs(lse - want_lse).max() <= 2e-3
    masks = np.stack([di.ancestor_mask_bits(x.parent[b], True) for b in range(cfg.batch)])
    assert masks.shape == (cfg.batch, 130, 3)
    got, _ = gu.run_verify(x, tree_mask=masks)
    assert np.array_equal(got, base)
    star = di.star_tree(cfg.n_tree)
    got2, _ = gu.run_verify(x, tree_mask=np.stack([di.ancestor_mask_bits(star, True)] * cfg.batch))
    want2, _ = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, np.stack([star] * cfg.batch), True)
    assert np.abs(got2 - want2).max() <= TOL["bf16"]
    # draft cross-attention: 10 query rows per call that name deep nodes of the wide tree (strict ancestors)
    xx = di.verify_inputs(cfg, prefix_len=[111, 60], streams=(di.STREAM_XQ, di.STREAM_XK, di.STREAM_XV))
    rows = np.stack([np.arange(120, 130, dtype=np.int32)] * cfg.batch)
    gotx, qsel = gu.run_xattn(xx, rows, rows)
    wantx, _ = oracle.tree_attn(qsel, xx.k, xx.v, "bf16", xx.prefix_len, xx.parent, False, q_node=rows)
    assert np.abs(gotx - wantx).max() <= TOL["bf16"]
    # float32 tensors
    cfg32 = _cfg("wide130_f32", "f32", 1, 2, 2, 64, 40, 9, 130, 9, 45)
    x32 = di.verify_inputs(cfg32)
    got32, _ = gu.run_verify(x32)
    want32, _ = oracle.tree_attn(x32.q, x32.k, x32.v, "f32", x32.prefix_len, x32.parent, True)
    assert np.abs(got32 - want32).max() <= TOL["f32"]


def test_seeded_random_shapes_with_the_automatic_plan(gu):
    """48 seeded shapes (batch, head grouping, head_dim, tree size, ragged prefix lengths incl. empty ones) through
    whatever kernel the launch plan picks, every element against the oracle; the set of plans reached is reported."""
    rng = np.random.default_rng(20250519)
    plans = set()
    for i in range(48):
        D = int(rng.choice([64, 128, 256]))
        hkv, g = [(1, 1), (2, 1), (2, 2), (2, 4), (4, 1), (8, 1), (3, 2)][int(rng.integers(7))]
        B = int(rng.integers(1, 6))
        T = int(rng.choice([1, 7, 16, 17, 33, 60, 64, 90]))
        depth = min(6, T - 1)
        prefix = int(rng.choice([0, 5, 31, 32, 100, 257, 700]))
        n_vis = (prefix * 3) // 4
        cfg = di.Config("rand%d" % i, "bf16", B, hkv * g, hkv, D, hkv * g * D, n_vis, prefix - n_vis, T, depth, 1, 4, 1000, 1, 200 + i)
        pl = [prefix] + [int(rng.integers(0, prefix + 1)) for _ in range(B - 1)]
        x = di.verify_inputs(cfg, prefix_len=pl)
        plans.add(gu.verify_plan(x).split(" ")[0])
        got, lse = gu.run_verify(x)
        want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
        assert np.isfinite(got).all(), (i, cfg)
        assert np.abs(got - want).max() <= TOL["bf16"], (i, cfg, np.abs(got - want).max())
        assert np.abs(lse - want_lse).max() <= 2e-3, (i, cfg)
    assert len(plans) >= 6, plans


def test_more_query_rows_than_tree_nodes(gu):
    """dream_draft_xattn with 100 query rows that name nodes of a 60-node tree (nodes repeat): every row against the oracle."""
    cfg = _cfg("manyrows", "bf16", 2, 4, 2, 128, 150, 43, 60, 6, 46)
    x = di.verify_inputs(cfg, prefix_len=[193, 80], streams=(di.STREAM_XQ, di.STREAM_XK, di.STREAM_XV))
    rng = np.random.default_rng(5)
    nodes = rng.integers(0, 60, size=(cfg.batch, 100)).astype(np.int32)
    got, qsel = gu.run_xattn(x, nodes, nodes)
    want, _ = oracle.tree_attn(qsel, x.k, x.v, "bf16", x.prefix_len, x.parent, False, q_node=nodes)
    assert np.abs(got - want).max() <= TOL["bf16"]


def test_custom_scale(gu):
    cfg = _cfg("scale", "bf16", 1, 4, 4, 64, 80, 20, 30, 5, 42)
    x = di.verify_inputs(cfg)
    got, _ = gu.run_verify(x, scale=0.05)
    want, _ = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True, scale=0.05)
    assert np.abs(got - want).max() <= TOL["bf16"]


def test_outputs_are_reproducible_bit_for_bit(gu):
    cfg = _cfg("repro", "bf16", 1, 8, 8, 128, 300, 60, 60, 6, 43)
    x = di.verify_inputs(cfg)
    dev = gu.DeviceAttn(x)
    a, la = gu.run_verify(x, dev=dev)
    b, lb = gu.run_verify(x, dev=dev)
    assert np.array_equal(a, b) and np.array_equal(la, lb)


@pytest.mark.parametrize("case", VARIANT_CASES + EXTRA_W8_CASES, ids=[c.variant for c in VARIANT_CASES] + ["extra-" + c.variant for c in EXTRA_W8_CASES])
def test_every_kernel_variant_all_elements(gu, case):
    """One case per bf16 kernel variant the launch plan can choose (tests/test_abi.py checks the list is complete):
    the plan must name that variant, and every output element and log-sum-exp must match the oracle."""
    import paper_2505_19201_amd as dream
    cfg = variant_config(case)
    x = di.verify_inputs(cfg, prefix_len=variant_prefix_lens(case))
    dream.dream_set_kv_splits(case.splits)
    dream.dream_set_q_tiles(case.q_tiles)
    dream.dream_set_tile_waves(case.waves)
    try:
        assert gu.verify_plan(x).startswith(case.variant + " "), gu.verify_plan(x)
        got, lse = gu.run_verify(x)
    finally:
        dream.dream_set_kv_splits(0)
        dream.dream_set_q_tiles(0)
        dream.dream_set_tile_waves(0)
    want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= TOL["bf16"], np.abs(got - want).max()
    assert np.abs(lse - want_lse).max() <= 2e-3


# shapes whose plans are the kernels that cut the work into query tiles and column slices, one per way of cutting: batch, heads, KV heads, head_dim, rows
SLICED = [(1, 32, 32, 128, 9), (2, 32, 32, 128, 60), (4, 32, 16, 128, 40), (4, 32, 32, 128, 60), (8, 32, 8, 128, 33), (2, 32, 32, 64, 17),
          (4, 32, 32, 64, 60), (1, 16, 8, 256, 60), (4, 16, 8, 256, 33), (4, 16, 8, 256, 60), (6, 16, 8, 256, 49)]


@pytest.mark.parametrize("shape", SLICED, ids=["x".join(map(str, x)) for x in SLICED])
def test_sliced_kernels_at_tile_edges(gu, shape):
    """Ranges around the 16- and 32-key tiles and around the number of key groups, sequences without a prefix beside full ones, a last query
    tile that is partly empty; and the same rows as a cross-attention call that names its nodes, under an explicit mask."""
    B, Hq, Hkv, D, T = shape
    plans = set()
    for prefix in (0, 15, 32 - T % 32, 128 - T, 129 - T, 256 - T, 257 - T):
        prefix = max(prefix, 0)
        cfg = _cfg("edge", "bf16", B, Hq, Hkv, D, prefix, 0, T, min(5, T - 1), 48)
        x = di.verify_inputs(cfg, prefix_len=[prefix if b % 3 != 1 else prefix // 2 for b in range(B)])
        plans.add(gu.verify_plan(x).split("<")[0])
        got, lse = gu.run_verify(x)
        want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
        assert np.isfinite(got).all(), prefix
        assert np.abs(got - want).max() <= TOL["bf16"], (prefix, np.abs(got - want).max())
        assert np.abs(lse - want_lse).max() <= 2e-3, prefix
    assert plans <= {"attn_wave_kernel", "attn_pair_kernel"}, plans
    star = np.stack([di.ancestor_mask_bits(di.star_tree(T), True)[:, 0]] * B)
    got, _ = gu.run_verify(x, tree_mask=star)
    want, _ = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, np.stack([di.star_tree(T)] * B), True)
    assert np.abs(got - want).max() <= TOL["bf16"]
    rows = np.stack([np.roll(np.arange(T, dtype=np.int32), 3)] * B)
    got, qsel = gu.run_xattn(x, rows, rows)
    want, _ = oracle.tree_attn(qsel, x.k, x.v, "bf16", x.prefix_len, x.parent, False, q_node=rows)
    assert np.abs(got - want).max() <= TOL["bf16"]


def test_two_slots_of_narrow_heads_at_tile_edges(gu):
    test_sliced_kernels_at_tile_edges(gu, (6, 32, 32, 64, 49))


@pytest.mark.parametrize("kv_len", [256, 257, 288, 511, 512, 513, 768, 1024, 1057, 1280, 1300, 2048])
def test_swapped_steps(gu, kv_len):
    """Two slices of heads of 64: odd workgroups swap the tiles of every two steps; one to eight steps, a last step without a partner, the tree and
    the ragged end in a tile that is taken ahead of an earlier one."""
    cfg = _cfg("swap", "bf16", 1, 32, 32, 64, kv_len - 60, 0, 60, 6, 51)
    x = di.verify_inputs(cfg)
    assert gu.verify_plan(x).startswith("attn_wave_kernel<64,8,2,1>"), gu.verify_plan(x)
    got, lse = gu.run_verify(x)
    want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
    assert np.abs(got - want).max() <= TOL["bf16"]
    assert np.abs(lse - want_lse).max() <= 2e-3


# one sequence and several ragged ones, two, four and one slices, one and more query tiles of several heads: batch, heads, KV heads, head_dim, rows, kernel,
# kv_lens (steps of all waves are 128 or 256 keys).  A last round of the order with one step, whole ones, the ragged end and the tree in a tile that is taken early; where the kernel serves ranges that long, three rounds.
TURNED = [
    (1, 32, 32, 128, 60, "attn_wave_kernel<128,8,2,1>", (128, 129, 256, 640, 1025, 1152, 1153, 1320)),
    (3, 32, 8, 128, 17, "attn_wave_kernel<128,8,2,1>", (128, 129, 256, 640, 1025, 1152, 1153, 1320, 2049)),
    (1, 32, 8, 128, 17, "attn_wave_kernel<128,8,4,1>", (256, 257, 512, 1025, 1280)),
    (2, 32, 32, 64, 33, "attn_wave_kernel<64,8,1,1>", (256, 257, 512, 1280, 2049, 2304)),
    (1, 16, 8, 256, 60, "attn_wave_kernel<256,4,4,1>", (128, 129, 256, 640, 1025, 1152, 1153, 1320)),
    (3, 16, 8, 256, 17, "attn_wave_kernel<256,8,4,2>", (128, 129, 256, 640, 1025, 1152, 1153, 1320)),
    (3, 16, 8, 256, 33, "attn_wave_kernel<256,8,4,3>", (128, 129, 256, 640, 1025, 1152, 1153, 1320)),
]


def _compare_verify(gu, x, parent=None, **kw):
    oracle.set_threads(16)
    try:
        got, lse = gu.run_verify(x, **kw)
        want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent if parent is None else parent, True)
    finally:
        oracle.set_threads(1)
    assert np.abs(got - want).max() <= TOL["bf16"] and np.abs(lse - want_lse).max() <= 2e-3


@pytest.mark.parametrize("B,Hq,Hkv,D,T,kernel,kv_lens", TURNED)
def test_turned_steps(gu, B, Hq, Hkv, D, T, kernel, kv_lens):
    """Workgroups that take their steps in turned order, the mask derived from the parents and an explicit one."""
    for kv_len in kv_lens:
        cfg = _cfg("turn", "bf16", B, Hq, Hkv, D, kv_len - T, 0, T, min(5, T - 1), 54)
        x = di.verify_inputs(cfg, prefix_len=[(kv_len - T) * (3 - b) // 3 for b in range(B)])
        assert gu.verify_plan(x).split(" ")[0] == kernel, (kv_len, gu.verify_plan(x))
        _compare_verify(gu, x)
        if kv_len in kv_lens[-2:]:
            star = di.star_tree(T)
            _compare_verify(gu, x, parent=np.stack([star] * B), tree_mask=np.stack([di.ancestor_mask_bits(star, True)[:, 0]] * B))


# verifications of three workgroups to a KV head or more, the last kv_len below 6 MB of keys and values an XCD: up to there the order is turned, above it is not and the caches are read with
# the nontemporal hint (but in four slices)
LINE = [(5, 16, 16, 64, 33, "attn_wave_kernel<64,8,1,1>", 2343), (5, 24, 8, 128, 17, "attn_wave_kernel<128,8,1,1>", 2343), (2, 32, 32, 128, 17, "attn_wave_kernel<128,8,2,1>", 1464),
        (2, 32, 32, 128, 10, "attn_wave_kernel<128,8,4,1>", 1464), (9, 8, 8, 256, 33, "attn_wave_kernel<256,4,1,1>", 651), (6, 8, 8, 256, 17, "attn_wave_kernel<256,4,2,1>", 976),
        (3, 16, 8, 256, 33, "attn_wave_kernel<256,8,4,3>", 1953)]


@pytest.mark.parametrize("B,Hq,Hkv,D,T,kernel,line", LINE)
def test_both_sides_of_the_turned_order(gu, B, Hq, Hkv, D, T, kernel, line):
    for kv_len in (line, line + 1):
        assert (-(-B * Hkv // 8) * kv_len * D * 4 < 6000000) == (kv_len == line)
        cfg = _cfg("line", "bf16", B, Hq, Hkv, D, kv_len - T, 0, T, min(5, T - 1), 58)
        x = di.verify_inputs(cfg, prefix_len=[(kv_len - T) * (B - b) // B for b in range(B)])
        assert gu.verify_plan(x).split(" ")[0] == kernel, (kv_len, gu.verify_plan(x))
        _compare_verify(gu, x)


SINGLE_LAUNCH = [c for c in VARIANT_CASES if "bf16" not in c.variant]


@pytest.mark.parametrize("case", SINGLE_LAUNCH, ids=[c.variant for c in SINGLE_LAUNCH])
@pytest.mark.parametrize("bound", [70, 127, 128, 129, 255, 256, 300])
def test_rows_behind_the_last_live_one_hold_anything(gu, case, bound):
    """NaN in every row of the caches behind the live ones, which the kernels may ask for before they know how many are live: max_kv_len on both sides of the first step of all waves
    (128 or 256 keys), sequences that end in it, without a prefix too, a capacity above."""
    prefix = [max(bound - case.n_tree, 0), 0, 9, max(bound - case.n_tree, 0) // 2] * case.batch
    cfg = _cfg("dead", "bf16", case.batch, case.n_q_heads, case.n_kv_heads, case.head_dim, 0, 0, case.n_tree, case.depth, 57)
    x = di.verify_inputs(cfg, prefix_len=prefix[:case.batch], slack_rows=200)
    assert gu.verify_plan(x).startswith(("attn_wave", "attn_pair", "attn_quad")), gu.verify_plan(x)
    dev = gu.DeviceAttn(x)
    for b in range(case.batch):
        for cache in (dev.k, dev.v):
            cache[b, :, int(x.prefix_len[b]) + case.n_tree:] = float("nan")
    oracle.set_threads(16)
    try:
        want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
    finally:
        oracle.set_threads(1)
    for dev.max_kv in (dev.max_kv, x.s_max):
        got, lse = gu.run_verify(x, dev=dev)
        assert np.abs(got - want).max() <= TOL["bf16"] and np.abs(lse - want_lse).max() <= 2e-3


@pytest.mark.parametrize("kv_len", [300, 513, 1024, 1300])
@pytest.mark.parametrize("B,T", [(2, 17), (3, 9)])
def test_swapped_steps_of_ragged_sequences_under_a_mask(gu, B, T, kv_len):
    """The same for sequences of different lengths, one of them without a prefix, and under an explicit mask: several pairs of steps, with and without
    a last one that has no partner."""
    cfg = _cfg("swap", "bf16", B, 32, 32, 64, kv_len - T, 0, T, 4, 53)
    x = di.verify_inputs(cfg, prefix_len=[kv_len - T, (kv_len - T) * 2 // 3, 0][:B])
    assert gu.verify_plan(x).startswith("attn_wave_kernel<64,8,2,1>"), gu.verify_plan(x)
    got, lse = gu.run_verify(x)
    want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
    assert np.abs(got - want).max() <= TOL["bf16"] and np.abs(lse - want_lse).max() <= 2e-3
    star = di.star_tree(T)
    got, _ = gu.run_verify(x, tree_mask=np.stack([di.ancestor_mask_bits(star, True)[:, 0]] * B))
    want, _ = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, np.stack([star] * B), True)
    assert np.abs(got - want).max() <= TOL["bf16"]


@pytest.mark.parametrize("B,Hq,Hkv,D,T", [(16, 32, 8, 128, 33), (12, 32, 8, 128, 60), (12, 16, 8, 256, 60), (9, 16, 8, 256, 49)])
def test_four_slots_at_tile_edges(gu, B, Hq, Hkv, D, T):
    """The same for four query slots: no, one, fewer and more steps than a key group has stages, a last workgroup with few query tiles; under a
    mask, and as a cross-attention call."""
    for prefix in (0, 32 - T % 32, 64 - T % 64, 128 - T, 129 - T, 256 - T, 257 - T, 333, 400):
        prefix = max(prefix, 0)
        cfg = _cfg("edge", "bf16", B, Hq, Hkv, D, prefix, 0, T, min(5, T - 1), 48)
        x = di.verify_inputs(cfg, prefix_len=[prefix if b % 3 != 1 else prefix // 2 for b in range(B)])
        assert gu.verify_plan(x).startswith("attn_quad_kernel"), gu.verify_plan(x)
        got, lse = gu.run_verify(x)
        want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
        assert np.isfinite(got).all(), prefix
        assert np.abs(got - want).max() <= TOL["bf16"], (prefix, np.abs(got - want).max())
        assert np.abs(lse - want_lse).max() <= 2e-3, prefix
    star = np.stack([di.ancestor_mask_bits(di.star_tree(T), True)[:, 0]] * B)
    got, _ = gu.run_verify(x, tree_mask=star)
    want, _ = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, np.stack([di.star_tree(T)] * B), True)
    assert np.abs(got - want).max() <= TOL["bf16"]
    rows = np.stack([np.roll(np.arange(T, dtype=np.int32), 3)] * B)
    got, qsel = gu.run_xattn(x, rows, rows)
    want, _ = oracle.tree_attn(qsel, x.k, x.v, "bf16", x.prefix_len, x.parent, False, q_node=rows)
    assert np.abs(got - want).max() <= TOL["bf16"]


@pytest.mark.parametrize("B,Hq,Hkv,T", [(20, 32, 8, 10), (32, 16, 8, 24), (17, 32, 8, 13)])
def test_two_slots_with_few_query_tiles(gu, B, Hq, Hkv, T):
    """One workgroup for a KV head's three or four query tiles: the second slot's last tile is empty or half full."""
    for kv_len in (T, 64, 65, 128, 160, 257, 700):
        cfg = _cfg("few", "bf16", B, Hq, Hkv, 128, kv_len - T, 0, T, min(4, T - 1), 60)
        x = di.verify_inputs(cfg, prefix_len=[(kv_len - T) // (1 + b % 3) for b in range(B)])
        assert gu.verify_plan(x).startswith("attn_pair_kernel<128,1,2> workgroups=%d " % (B * Hkv)), gu.verify_plan(x)
        got, lse = gu.run_verify(x)
        oracle.set_threads(16)
        try:
            want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
        finally:
            oracle.set_threads(1)
        assert np.abs(got - want).max() <= TOL["bf16"] and np.abs(lse - want_lse).max() <= 2e-3, kv_len


@pytest.mark.parametrize("B,Hq,Hkv,T", [(5, 32, 32, 16), (8, 32, 32, 7), (13, 16, 16, 10), (30, 16, 8, 8)])
def test_one_query_tile_of_every_head_unsliced(gu, B, Hq, Hkv, T):
    """More KV heads than two slices leave CUs for, one query tile each: no, fewer and more steps than waves, with four waves and with eight."""
    for kv_len in (T, 32, 33, 160, 161, 256, 257, 700):
        cfg = _cfg("one", "bf16", B, Hq, Hkv, 128, kv_len - T, 0, T, min(4, T - 1), 59)
        x = di.verify_inputs(cfg, prefix_len=[(kv_len - T) // (1 + b % 3) for b in range(B)])
        assert re.match("attn_wave_kernel<128,[48],1,1> workgroups=%d " % (B * Hkv), gu.verify_plan(x)), gu.verify_plan(x)
        got, lse = gu.run_verify(x)
        oracle.set_threads(16)
        try:
            want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
        finally:
            oracle.set_threads(1)
        assert np.abs(got - want).max() <= TOL["bf16"] and np.abs(lse - want_lse).max() <= 2e-3, kv_len


@pytest.mark.parametrize("kernel,B,Hq,Hkv,D,T", [("wave", 3, 20, 5, 128, 17), ("wave", 2, 15, 5, 64, 33), ("wave", 7, 12, 12, 64, 9), ("wave", 5, 8, 4, 256, 33), ("wave", 33, 4, 1, 128, 16),
                                                 ("pair", 13, 16, 4, 128, 33), ("pair", 23, 20, 5, 128, 17), ("quad", 25, 20, 5, 128, 33), ("quad", 23, 8, 4, 256, 60)])
def test_kv_heads_that_do_not_fill_the_xcds(gu, kernel, B, Hq, Hkv, D, T):
    """KV heads and sequences are numbered together over the XCDs: counts that are no multiple of 8, ragged sequences."""
    assert B * Hkv % 8
    cfg = _cfg("odd", "bf16", B, Hq, Hkv, D, 740 - T, 0, T, 4, 57)
    x = di.verify_inputs(cfg, prefix_len=[(740 - T) // (1 + b % 4) for b in range(B)])
    assert gu.verify_plan(x).startswith("attn_%s_kernel" % kernel), gu.verify_plan(x)
    got, lse = gu.run_verify(x)
    oracle.set_threads(16)
    try:
        want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
    finally:
        oracle.set_threads(1)
    assert np.abs(got - want).max() <= TOL["bf16"] and np.abs(lse - want_lse).max() <= 2e-3


@pytest.mark.parametrize("shape,kv_len", [((2, 32, 32, 128, 9), 1984), ((1, 32, 32, 64, 9), 2016), ((1, 32, 8, 128, 64), 2688), ((2, 24, 8, 128, 33), 1568), ((8, 16, 8, 256, 9), 2304),
                                          ((3, 32, 32, 64, 9), 3840), ((24, 32, 8, 128, 17), 736), ((24, 32, 8, 128, 17), 737)])
def test_the_longest_ranges_of_single_launches(gu, shape, kv_len):
    """Ragged sequences at the lengths up to which a shape takes one launch without key splits (and from which it takes four slots)."""
    B, Hq, Hkv, D, T = shape
    cfg = _cfg("long", "bf16", B, Hq, Hkv, D, kv_len - T, 0, T, min(5, T - 1), 52)
    x = di.verify_inputs(cfg, prefix_len=[(kv_len - T) // (1 + b % 3) for b in range(B)])
    plan = gu.verify_plan(x)
    assert "splits=1 " in plan and (kv_len == 736 or not plan.startswith("attn_bf16")), plan
    got, lse = gu.run_verify(x)
    oracle.set_threads(16)
    try:
        want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
    finally:
        oracle.set_threads(1)
    assert np.abs(got - want).max() <= TOL["bf16"] and np.abs(lse - want_lse).max() <= 2e-3


def test_tensors_off_16_byte_boundaries_take_another_kernel(gu):
    """Loads straight to LDS need 16-byte aligned tensors: queries or caches that start elsewhere give the same rows within rounding, in
    the workspace the query returned."""
    import torch
    import paper_2505_19201_amd as dream
    cfg = _cfg("shifted", "bf16", 1, 32, 32, 128, 150, 43, 60, 6, 49)
    x = di.verify_inputs(cfg)
    assert gu.verify_plan(x).startswith("attn_wave_kernel")
    base, _ = gu.run_verify(x)
    for name in ("q", "k", "v"):
        dev = gu.DeviceAttn(x)
        t = getattr(dev, name)
        flat = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
        shifted = flat[2:2 + t.numel()].view(t.shape)
        shifted.copy_(t)
        assert shifted.data_ptr() % 16 == 4
        setattr(dev, name, shifted)
        got, _ = gu.run_verify(x, dev=dev)
        assert np.abs(got - base).max() <= TOL["bf16"], name


@pytest.mark.parametrize("B,Hq,Hkv,D,T,kernel", [(8, 32, 8, 128, 60, "attn_pair_kernel"), (16, 32, 8, 128, 60, "attn_quad_kernel"), (4, 16, 8, 256, 33, "attn_wave_kernel"),
                                                    (1, 32, 32, 128, 60, "attn_wave_kernel")])
def test_rows_leave_the_same_wherever_the_output_starts(gu, B, Hq, Hkv, D, T, kernel):
    """The few-stream kernels store 16 bytes a lane, whatever the output's alignment: the same bits, nothing beside the rows."""
    import torch
    import paper_2505_19201_amd as dream
    cfg = _cfg("out", "bf16", B, Hq, Hkv, D, 200, 43, T, 6, 60)
    x = di.verify_inputs(cfg, prefix_len=[243 - 9 * (b % 5) for b in range(B)])
    assert gu.verify_plan(x).startswith(kernel)
    base, _ = gu.run_verify(x)
    dev = gu.DeviceAttn(x)
    n = base.size
    desc = dream.attn_desc(B, Hq, Hkv, D, dream.BF16, dev.k.shape[2])
    ws = dream.alloc_workspace(dream.dream_tree_verify_attn_workspace(desc, T, dev.max_kv))
    for off in (2, 1):
        flat = torch.full((n + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
        out = flat[off:off + n].view(base.shape)
        assert out.data_ptr() % 16 == 2 * off
        dream.dream_tree_verify_attn(desc, dev.q, dev.k, dev.v, dev.prefix_len, T, dev.parent, None, dev.max_kv, out, None, ws)
        assert np.array_equal(out.float().cpu().numpy(), base.astype(np.float32))
        assert (flat[:off] == 7.0).all() and (flat[off + n:] == 7.0).all()


@pytest.mark.parametrize("B,Hq,Hkv,D,line", [(1, 32, 32, 128, 90), (2, 16, 8, 128, 100), (1, 32, 32, 64, 112), (2, 16, 8, 256, 72), (3, 24, 8, 128, 152), (3, 16, 16, 64, 112),
                                                  (3, 32, 32, 64, 60)])      # (the last: more keys than an XCD's L2 holds, steps in their own order)
def test_long_ranges_of_a_draft_cache(gu, B, Hq, Hkv, D, line):
    """Cross-attention over a cache that the memory-side cache holds stays one launch for longer than the plan of a verification says: lengths where the two differ,
    the last of them and the next, ragged sequences; a cache off the 16-byte boundaries in the workspace that the query returned."""
    import torch
    for kv_len in ((line - 11) * 32, line * 32, line * 32 + 1):
        cfg = _cfg("near", "bf16", B, Hq, Hkv, D, kv_len - 17, 0, 17, 4, 58)
        x = di.verify_inputs(cfg, prefix_len=[(kv_len - 17) // (1 + b) for b in range(B)], streams=(di.STREAM_XQ, di.STREAM_XK, di.STREAM_XV))
        rows = np.stack([np.arange(6, 16, dtype=np.int32)] * B)
        got, qsel = gu.run_xattn(x, rows, rows)
        oracle.set_threads(16)
        try:
            want, _ = oracle.tree_attn(qsel, x.k, x.v, "bf16", x.prefix_len, x.parent, False, q_node=rows)
        finally:
            oracle.set_threads(1)
        assert np.abs(got - want).max() <= TOL["bf16"], kv_len
    dev = gu.DeviceAttn(x)
    flat = torch.empty(dev.k.numel() + 8, dtype=dev.k.dtype, device="cuda")
    shifted = flat[2:2 + dev.k.numel()].view(dev.k.shape)
    shifted.copy_(dev.k)
    dev.k = shifted
    got, _ = gu.run_xattn(x, rows, rows, dev=dev)
    assert np.abs(got - want).max() <= TOL["bf16"]


FULL = ["llava", "pixtral", "gemma3", "smolvlm_b1", "smolvlm_b8", "smolvlm_b32"]


@pytest.mark.parametrize("name", FULL)
def test_full_size_verify_all_elements(gu, name):
    """Full measurement shape in the launch configuration bench.py times (asserted by its plan string): every output
    element and every log-sum-exp against the oracle (16 host threads)."""
    cfg = di.CONFIGS[name]
    x = di.verify_inputs(cfg)
    assert gu.verify_plan(x) == FULL_VERIFY_PLANS[name]
    got, lse = gu.run_verify(x)
    oracle.set_threads(16)
    try:
        want, want_lse = oracle.tree_attn(x.q, x.k, x.v, cfg.dtype, x.prefix_len, x.parent, True)
    finally:
        oracle.set_threads(1)
    assert np.isfinite(got).all() and np.isfinite(lse).all()
    assert np.abs(got - want).max() <= TOL["bf16"], np.abs(got - want).max()
    assert np.abs(lse - want_lse).max() <= 2e-3


# ------------------------------------------------------------------------------------------------
# draft cross-attention: strict ancestors, one call per tree level
# ------------------------------------------------------------------------------------------------
def test_tiny_config_xattn_levels(gu):
    cfg = di.CONFIGS["tiny"]
    x = di.xattn_inputs(cfg)
    for lv in di.tree_levels(x.parent[0]):
        rows = lv[None]
        got, qsel = gu.run_xattn(x, rows, rows)
        want, _ = oracle.tree_attn(qsel, x.k, x.v, cfg.dtype, x.prefix_len, x.parent, False, q_node=rows)
        assert np.abs(got - want).max() <= TOL["f32"]


XCASES = [
    ("x_mha128", 2, 4, 4, 128, 150, 43, 60, 6, [193, 101]),
    ("x_gqa4_128", 1, 8, 2, 128, 130, 31, 60, 6, [161]),
    ("x_gqa2_256", 1, 4, 2, 256, 120, 45, 60, 6, [165]),
    ("x_mha64", 2, 4, 4, 64, 200, 57, 60, 6, [257, 130]),
]


@pytest.mark.parametrize("case", XCASES, ids=[c[0] for c in XCASES])
def test_bf16_xattn_levels_all_elements(gu, case):
    name, B, Hq, Hkv, D, v, q, T, depth, pl = case
    cfg = _cfg(name, "bf16", B, Hq, Hkv, D, v, q, T, depth, 44)
    x = di.verify_inputs(cfg, prefix_len=pl, streams=(di.STREAM_XQ, di.STREAM_XK, di.STREAM_XV))
    dev = gu.DeviceAttn(x)
    for lvl in range(depth + 1):
        rows = np.stack([di.tree_levels(x.parent[b])[lvl] for b in range(B)])
        got, qsel = gu.run_xattn(x, rows, rows, dev=dev)
        want, _ = oracle.tree_attn(qsel, x.k, x.v, "bf16", x.prefix_len, x.parent, False, q_node=rows)
        assert np.abs(got - want).max() <= TOL["bf16"]


def test_xattn_all_nodes_in_one_call_without_q_node(gu):
    cfg = _cfg("x_all", "bf16", 1, 4, 4, 128, 100, 28, 60, 6, 45)
    x = di.verify_inputs(cfg)
    rows = np.arange(cfg.n_tree, dtype=np.int32)[None]
    got, qsel = gu.run_xattn(x, rows, None)
    want, _ = oracle.tree_attn(qsel, x.k, x.v, "bf16", x.prefix_len, x.parent, False)
    assert np.abs(got - want).max() <= TOL["bf16"]
    # strict mask differs from the verification mask
    ver, _ = oracle.tree_attn(qsel, x.k, x.v, "bf16", x.prefix_len, x.parent, True)
    assert np.abs(got - ver).max() > 1e-3


def test_xattn_root_with_empty_prefix_gives_zero_row(gu):
    cfg = _cfg("x_empty", "bf16", 1, 2, 2, 64, 0, 0, 12, 3, 46)
    x = di.verify_inputs(cfg, prefix_len=[0])
    rows = np.arange(cfg.n_tree, dtype=np.int32)[None]
    got, qsel = gu.run_xattn(x, rows, rows)
    want, _ = oracle.tree_attn(qsel, x.k, x.v, "bf16", x.prefix_len, x.parent, False, q_node=rows)
    assert np.all(got[0, 0] == 0.0)
    assert np.abs(got - want).max() <= TOL["bf16"]


@pytest.mark.parametrize("name", FULL)
def test_full_size_xattn_round_all_elements(gu, name):
    """One drafting round at the measurement shape: a call per tree level (1,10,10,10,10,10,9 rows), in the launch
    configuration bench.py times (asserted by the plan strings); every output element against the oracle."""
    cfg = di.CONFIGS[name]
    x = di.xattn_inputs(cfg)
    dev = gu.DeviceAttn(x)
    root_plan, level_plan = FULL_XATTN_PLANS[name]
    oracle.set_threads(16)
    try:
        for lvl in range(cfg.depth + 1):
            rows = np.stack([di.tree_levels(x.parent[b])[lvl] for b in range(cfg.batch)])
            if rows.shape[1] in (1, 10):
                assert gu.xattn_plan(x, rows.shape[1]) == (root_plan if rows.shape[1] == 1 else level_plan)
            got, qsel = gu.run_xattn(x, rows, rows, dev=dev)
            want, _ = oracle.tree_attn(qsel, x.k, x.v, cfg.dtype, x.prefix_len, x.parent, False, q_node=rows)
            assert np.isfinite(got).all()
            assert np.abs(got - want).max() <= TOL["bf16"], (lvl, np.abs(got - want).max())
    finally:
        oracle.set_threads(1)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_malformed_device_metadata_stays_in_bounds(gu, dtype):
    """A prefix length past the cache and a parent array with cycles give unspecified numbers but finite ones:
    the kernels clamp the prefix to the cache and treat a parent that does not precede its node as none."""
    cfg = di.Config("bad_meta", dtype, 1, 4, 2, 64, 256, 40, 24, 12, 4, 1, 4, 64, 1, 31)
    x = di.verify_inputs(cfg)
    good, _ = gu.run_verify(x)
    dev = gu.DeviceAttn(x)
    par = x.parent.copy()
    par[0, 3], par[0, 5], par[0, 6], par[0, 7] = 3, 6, 5, 99
    dev.parent = dream_to_device(par)
    dev.prefix_len = dream_to_device(np.array([x.s_max + 1000], dtype=np.int32))
    dev.max_kv = x.s_max
    got, lse = gu.run_verify(x, dev=dev)
    assert np.isfinite(got).all() and np.isfinite(lse).all()
    dev.prefix_len = dream_to_device(np.array([-17], dtype=np.int32))       # clamps to an empty prefix
    got, _ = gu.run_verify(x, dev=dev)
    assert np.isfinite(got).all()
    again, _ = gu.run_verify(x)                                             # and the well-formed call is unaffected
    assert np.array_equal(good, again)


def dream_to_device(a):
    import paper_2505_19201_amd as dream
    return dream.to_device(a)


@pytest.mark.parametrize("D,kv", [(D, kv) for D in (64, 128, 256) for kv in (9, 31, 32, 33, 64, 65, 127, 128, 129, 300)])
def test_f32_pass_edges(gu, D, kv):
    """Key counts around the float32 kernel's passes (128, 64 and 32 keys at head_dim 64, 128 and 256), grouped queries, one
    sequence shorter than the other."""
    T = 9
    cfg = _cfg("f32edge", "f32", 2, 4, 2, D, kv - T, 0, T, 4, 46)
    x = di.verify_inputs(cfg, prefix_len=[kv - T, (kv - T) // 2])
    got, lse = gu.run_verify(x)
    want, want_lse = oracle.tree_attn(x.q, x.k, x.v, "f32", x.prefix_len, x.parent, True)
    assert np.abs(got - want).max() <= TOL["f32"] and np.abs(lse - want_lse).max() <= 1e-5


@pytest.mark.parametrize("shape", [(8, 32, 32, 128, 1300), (16, 32, 8, 128, 2500)])
def test_levels_over_a_cache_beyond_the_memory_side_cache(gu, shape):
    """Cross-attention reads caches of more than 152 MB with the nontemporal hint."""
    B, Hq, Hkv, D, prefix = shape
    assert B * Hkv * (prefix + 17) * D * 4 >= 152 << 20
    cfg = _cfg("large", "bf16", B, Hq, Hkv, D, prefix, 0, 17, 4, 54)
    x = di.verify_inputs(cfg, prefix_len=[prefix - 61 * b for b in range(B)], streams=(di.STREAM_XQ, di.STREAM_XK, di.STREAM_XV))
    rows = np.stack([np.arange(5, 9, dtype=np.int32)] * B)
    assert gu.xattn_plan(x, 4).startswith("attn_wave_kernel"), gu.xattn_plan(x, 4)
    got, qsel = gu.run_xattn(x, rows, rows)
    want, _ = oracle.tree_attn(qsel, x.k, x.v, "bf16", x.prefix_len, x.parent, False, q_node=rows)
    assert np.abs(got - want).max() <= TOL["bf16"]
