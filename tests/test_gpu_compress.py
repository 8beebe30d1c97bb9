"""GPU parity: dream_visual_compress.  Stage B (top-k keep) is bit-exact on identical float32 scores;
stage A scores are compared to the float64 oracle; end-to-end kept indices are bit-exact on seeds whose
k-th / (k+1)-th oracle scores are separated by more than the float32 evaluation error (the seed is
screened on the oracle side only, before the GPU result is looked at)."""
import numpy as np
import pytest

import dream_inputs as di
import oracle

pytestmark = pytest.mark.gpu

GAP = 1e-4      # minimum relative gap between the k-th and (k+1)-th oracle score for an end-to-end index check
SCORE_RTOL = {"f32": 2e-5, "bf16": 2e-4}


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from tests import gpu_util
    return gpu_util


def _qk(cfg, seed, n_q=None, extra_rows=3):
    q = di.prefill_q(cfg, n_q, seed)
    k = di.normal((cfg.batch, cfg.n_kv_heads, cfg.prefix + extra_rows, cfg.head_dim), cfg.dtype, seed, di.STREAM_K)
    return q, k


def _boundary_gap(scores64, k):
    """Smallest relative gap over the batch between the last kept and the first dropped score."""
    worst = np.inf
    for row in scores64:
        s = np.sort(row)[::-1]
        if 0 < k < len(s):
            worst = min(worst, (s[k - 1] - s[k]) / abs(s[k - 1]))
    return worst


def _pick_seed(cfg, vis_start, vis_len, q_pos=None):
    """First seed of a fixed list whose oracle scores have a safe gap at the keep boundary."""
    k = oracle.keep_count(vis_len, cfg.keep_num, cfg.keep_den)
    for seed in [cfg.seed + 1000 * i for i in range(5)]:
        q, kk = _qk(cfg, seed)
        want = oracle.visual_scores(q, kk, cfg.dtype, vis_start, vis_len, q_pos=q_pos)
        if _boundary_gap(want, k) > GAP:
            return seed, q, kk, want
    raise AssertionError("no seed with a safe top-k boundary")


def test_stage_b_is_bit_exact_on_given_scores(gu):
    g = di.rng(11, di.STREAM_SCORES)
    cases = [(1, 1, 1, 2), (3, 5, 1, 2), (2, 64, 1, 4), (2, 576, 1, 4), (4, 1088, 1, 4), (1, 1025, 3, 4), (2, 2500, 1, 3),
             (1, 16384, 1, 4), (2, 37, 0, 1), (2, 37, 1, 1)]
    for (B, v, num, den) in cases:
        s = g.standard_normal(size=(B, v), dtype=np.float32)
        s[:, ::3] = np.float32(0.5)                               # a third of the entries tie exactly
        s[0, : v // 2] = np.round(s[0, : v // 2] * 2) / 2          # coarse values: many more ties
        _, kept, _ = gu.run_compress("bf16", None, None, 0, 7, v, num, den, scores_in=s)
        want = oracle.topk_keep(s, 7, num, den)
        assert np.array_equal(kept, want), (B, v, num, den)


def test_tiny_config_scores_kept_and_gather(gu):
    cfg = di.CONFIGS["tiny"]
    seed, q, k, want = _pick_seed(cfg, 0, cfg.n_visual)
    rows = di.feature_rows(cfg, seed=seed)
    scores, kept, gathered = gu.run_compress(cfg.dtype, q, k, cfg.prefix, 0, cfg.n_visual, cfg.keep_num, cfg.keep_den,
                                             gather_src=rows)
    np.testing.assert_allclose(scores, want, rtol=SCORE_RTOL["f32"])
    want_kept = oracle.topk_keep(want, 0, cfg.keep_num, cfg.keep_den)
    assert kept.shape == (1, 32) and np.array_equal(kept, want_kept)
    assert np.array_equal(gathered, oracle.gather_rows(rows, cfg.dtype, want_kept))
    # stage B alone on the GPU's own float32 scores
    assert np.array_equal(kept, oracle.topk_keep(scores, 0, cfg.keep_num, cfg.keep_den))


SMALL = [
    # name, B, Hq, Hkv, D, v, q_text, vis_start, keep
    ("mha128", 2, 4, 4, 128, 150, 43, 0, (1, 4)),
    ("gqa4_128_offset", 1, 8, 2, 128, 130, 61, 20, (1, 2)),
    ("gqa2_256", 1, 4, 2, 256, 100, 37, 5, (3, 4)),
    ("mha64", 2, 4, 4, 64, 200, 57, 9, (1, 4)),
]


@pytest.mark.parametrize("case", SMALL, ids=[c[0] for c in SMALL])
def test_bf16_scores_and_kept_small(gu, case):
    name, B, Hq, Hkv, D, v, qt, vs, (num, den) = case
    cfg = di.Config(name, "bf16", B, Hq, Hkv, D, 64, v, qt, 8, 3, num, den, 100, 1, 60)
    seed, q, k, want = _pick_seed(cfg, vs, v)
    rows = di.feature_rows(cfg, seed=seed)
    scores, kept, gathered = gu.run_compress("bf16", q, k, cfg.prefix, vs, v, num, den, gather_src=rows)
    np.testing.assert_allclose(scores, want, rtol=SCORE_RTOL["bf16"])
    want_kept = oracle.topk_keep(want, vs, num, den)
    assert np.array_equal(kept, want_kept)
    assert np.array_equal(kept, oracle.topk_keep(scores, vs, num, den))
    assert np.array_equal(gathered, oracle.gather_rows(rows, "bf16", want_kept))


def test_explicit_row_positions(gu):
    cfg = di.Config("pos", "bf16", 2, 4, 2, 128, 64, 90, 30, 8, 3, 1, 2, 100, 1, 61)
    P = cfg.prefix
    n_q = 50
    pos = np.stack([np.sort(di.rng(5, 903, b).permutation(P)[:n_q])[::-1] for b in range(cfg.batch)]).astype(np.int32)
    q = di.prefill_q(cfg, n_q, 8)
    k = di.normal((cfg.batch, cfg.n_kv_heads, P + 2, cfg.head_dim), "bf16", 8, di.STREAM_K)
    want = oracle.visual_scores(q, k, "bf16", 10, 80, q_pos=pos)
    scores, kept, _ = gu.run_compress("bf16", q, k, P, 10, 80, 1, 2, q_pos=pos)
    np.testing.assert_allclose(scores, want, rtol=SCORE_RTOL["bf16"], atol=1e-6)
    assert np.array_equal(kept, oracle.topk_keep(scores, 10, 1, 2))


def test_scores_are_reproducible_bit_for_bit(gu):
    cfg = di.Config("rep", "bf16", 1, 8, 8, 128, 64, 300, 84, 8, 3, 1, 4, 100, 1, 62)
    q, k = _qk(cfg, 3)
    a, ka, _ = gu.run_compress("bf16", q, k, cfg.prefix, 0, 300, 1, 4)
    b, kb, _ = gu.run_compress("bf16", q, k, cfg.prefix, 0, 300, 1, 4)
    assert np.array_equal(a, b) and np.array_equal(ka, kb)


def test_zero_keep_and_zero_span(gu):
    cfg = di.Config("z", "bf16", 1, 4, 4, 64, 64, 40, 10, 8, 3, 0, 1, 100, 1, 63)
    q, k = _qk(cfg, 4)
    scores, kept, _ = gu.run_compress("bf16", q, k, cfg.prefix, 0, 40, 0, 1)
    assert kept.shape == (1, 0) and np.isfinite(scores).all()
    scores, kept, _ = gu.run_compress("bf16", q, k, cfg.prefix, 0, 0, 1, 2, want_scores=False)
    assert kept.shape == (1, 0)


@pytest.mark.parametrize("name", ["llava", "pixtral", "gemma3", "smolvlm_b1", "smolvlm_b8"])
def test_full_size_configs(gu, name):
    """Measurement shapes, all prefill rows: scores against the oracle, kept indices and gathered rows
    bit-exact (seed screened for a safe boundary gap on the oracle side)."""
    cfg = di.CONFIGS[name]
    oracle.set_threads(min(16, oracle.hw_threads()))
    try:
        seed, q, k, want = _pick_seed(cfg, 0, cfg.n_visual)
    finally:
        oracle.set_threads(1)
    rows = di.feature_rows(cfg, seed=seed)
    scores, kept, gathered = gu.run_compress("bf16", q, k, cfg.prefix, 0, cfg.n_visual, cfg.keep_num, cfg.keep_den,
                                             gather_src=rows)
    np.testing.assert_allclose(scores, want, rtol=SCORE_RTOL["bf16"])
    want_kept = oracle.topk_keep(want, 0, cfg.keep_num, cfg.keep_den)
    assert kept.shape[1] == oracle.keep_count(cfg.n_visual, cfg.keep_num, cfg.keep_den)
    assert np.array_equal(kept, want_kept)
    assert np.array_equal(kept, oracle.topk_keep(scores, 0, cfg.keep_num, cfg.keep_den))
    assert np.array_equal(gathered, oracle.gather_rows(rows, "bf16", want_kept))


def test_full_size_smolvlm_b32(gu):
    """32 sequences per call, all prefill rows.  Scores of every sequence against the oracle; the kept set is the exact
    top-k of the library's own float32 scores for every sequence, and equals the oracle's kept set wherever the
    oracle's boundary gap is safe (decided per sequence on the oracle side; most sequences must qualify)."""
    cfg = di.CONFIGS["smolvlm_b32"]
    q, k = _qk(cfg, cfg.seed)
    oracle.set_threads(min(16, oracle.hw_threads()))
    try:
        want = oracle.visual_scores(q, k, cfg.dtype, 0, cfg.n_visual)
    finally:
        oracle.set_threads(1)
    n_keep = oracle.keep_count(cfg.n_visual, cfg.keep_num, cfg.keep_den)
    safe = np.array([_boundary_gap(want[b:b + 1], n_keep) > GAP for b in range(cfg.batch)])
    assert safe.sum() >= cfg.batch // 2
    rows = di.feature_rows(cfg)
    scores, kept, gathered = gu.run_compress("bf16", q, k, cfg.prefix, 0, cfg.n_visual, cfg.keep_num, cfg.keep_den, gather_src=rows)
    np.testing.assert_allclose(scores, want, rtol=SCORE_RTOL["bf16"])
    assert np.array_equal(kept, oracle.topk_keep(scores, 0, cfg.keep_num, cfg.keep_den))
    want_kept = oracle.topk_keep(want, 0, cfg.keep_num, cfg.keep_den)
    assert np.array_equal(kept[safe], want_kept[safe])
    assert np.array_equal(gathered, oracle.gather_rows(rows, "bf16", kept))


def _causal_row_lse(q, k, dtype, scale=None, q_pos=None):
    """Natural-log sum of exp of the scaled scores of every row over keys 0..pos(row), float64 numpy: [B, Hq, n_q].
    (What an attention kernel with a log-sum-exp output leaves; written out here so that nothing comes from the GPU.)"""
    qf, kf = di.as_f64(q, dtype), di.as_f64(k, dtype)
    B, n_q, Hq, D = qf.shape
    Hkv = kf.shape[1]
    scale = 1.0 / np.sqrt(D) if scale is None else scale
    out = np.empty((B, Hq, n_q))
    for b in range(B):
        pos = np.arange(n_q) if q_pos is None else np.asarray(q_pos)[b]
        for h in range(Hq):
            s = qf[b, :, h, :] @ kf[b, h // (Hq // Hkv)].T * scale            # [n_q, n_keys]
            s = np.where(np.arange(s.shape[1])[None, :] <= pos[:, None], s, -np.inf)
            m = s.max(axis=1)
            out[b, h] = m + np.log(np.exp(s - m[:, None]).sum(axis=1))
    return out


@pytest.mark.parametrize("case", SMALL, ids=[c[0] for c in SMALL])
def test_caller_supplied_row_lse_small(gu, case):
    """With the rows' log-sum-exps given, stage A is one pass: same scores (to tolerance) and the same kept set."""
    name, B, Hq, Hkv, D, v, qt, vs, (num, den) = case
    cfg = di.Config(name, "bf16", B, Hq, Hkv, D, 64, v, qt, 8, 3, num, den, 100, 1, 60)
    seed, q, k, want = _pick_seed(cfg, vs, v)
    lse = _causal_row_lse(q, k, "bf16")
    scores, kept, _ = gu.run_compress("bf16", q, k, cfg.prefix, vs, v, num, den, row_lse=lse)
    np.testing.assert_allclose(scores, want, rtol=SCORE_RTOL["bf16"])
    assert np.array_equal(kept, oracle.topk_keep(want, vs, num, den))


def test_caller_supplied_row_lse_tiny_f32_and_positions(gu):
    cfg = di.CONFIGS["tiny"]
    seed, q, k, want = _pick_seed(cfg, 0, cfg.n_visual)
    lse = _causal_row_lse(q, k, "f32")
    scores, kept, _ = gu.run_compress("f32", q, k, cfg.prefix, 0, cfg.n_visual, cfg.keep_num, cfg.keep_den, row_lse=lse)
    np.testing.assert_allclose(scores, want, rtol=SCORE_RTOL["f32"])
    assert np.array_equal(kept, oracle.topk_keep(want, 0, cfg.keep_num, cfg.keep_den))
    # explicit, shuffled row positions (bf16)
    c2 = di.Config("pos_lse", "bf16", 2, 4, 2, 128, 512, 100, 60, 8, 3, 1, 2, 100, 1, 62)
    q, k = _qk(c2, 5, n_q=90)
    g = di.rng(63, 902)
    q_pos = np.stack([g.permutation(c2.prefix)[:90] for _ in range(c2.batch)]).astype(np.int32)
    want = oracle.visual_scores(q, k, "bf16", 10, 80, q_pos=q_pos)
    lse = _causal_row_lse(q, k, "bf16", q_pos=q_pos)
    scores, kept, _ = gu.run_compress("bf16", q, k, c2.prefix, 10, 80, 1, 2, q_pos=q_pos, row_lse=lse)
    np.testing.assert_allclose(scores, want, rtol=SCORE_RTOL["bf16"])


@pytest.mark.parametrize("name", ["llava", "gemma3"])
def test_caller_supplied_row_lse_full_size(gu, name):
    cfg = di.CONFIGS[name]
    oracle.set_threads(min(16, oracle.hw_threads()))
    try:
        seed, q, k, want = _pick_seed(cfg, 0, cfg.n_visual)
    finally:
        oracle.set_threads(1)
    lse = _causal_row_lse(q, k, "bf16")
    scores, kept, _ = gu.run_compress("bf16", q, k, cfg.prefix, 0, cfg.n_visual, cfg.keep_num, cfg.keep_den, row_lse=lse)
    np.testing.assert_allclose(scores, want, rtol=SCORE_RTOL["bf16"])
    assert np.array_equal(kept, oracle.topk_keep(want, 0, cfg.keep_num, cfg.keep_den))


@pytest.mark.parametrize("v", [63, 64, 65, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049])
@pytest.mark.parametrize("num,den", [(1, 4), (1, 1), (1, 97)])
def test_selection_sizes_and_ties(gu, v, num, den):
    """Token counts around the selection kernels' register files, scores with many exact ties and of both signs."""
    g = di.rng(17 + v, di.STREAM_SCORES)
    s = np.round(g.standard_normal(size=(3, v)).astype(np.float32) * 3) / 3
    s[1] = g.standard_normal(size=v)
    s[2] = np.float32(0.25)                                      # everything ties: the first k tokens
    _, kept, _ = gu.run_compress("bf16", None, None, 0, 3, v, num, den, scores_in=s)
    assert np.array_equal(kept, oracle.topk_keep(s, 3, num, den))


@pytest.mark.parametrize("D,P,v,vis_start,with_pos", [(64, 1, 1, 0, False), (64, 63, 40, 7, False), (128, 65, 64, 1, False), (128, 129, 65, 63, False),
                                                      (256, 257, 130, 64, False), (64, 700, 600, 50, True), (64, 1300, 1200, 0, False)])
def test_score_steps_and_splits(gu, D, P, v, vis_start, with_pos):
    """Rows and keys around the 64-row steps, blocks with different numbers of splits, more rows than one window of log-sum-exps."""
    H = 2
    g = di.rng(1000 + P, di.STREAM_SCORES)
    q = di.normal((2, P, H, D), "bf16", 1001 + P, di.STREAM_PREFILL_Q)
    k = di.normal((2, H, P + 3, D), "bf16", 1002 + P, di.STREAM_K)
    pos = np.stack([g.permutation(P) for _ in range(2)]).astype(np.int32) if with_pos else None
    scores, _, _ = gu.run_compress("bf16", q, k, P, vis_start, v, 1, 2, q_pos=pos)
    np.testing.assert_allclose(scores, oracle.visual_scores(q, k, "bf16", vis_start, v, q_pos=pos), rtol=SCORE_RTOL["bf16"])


@pytest.mark.parametrize("B,H,D,P,v,vis_start,with_pos", [(2, 16, 64, 700, 640, 9, False), (2, 8, 64, 1279, 1100, 0, False), (3, 7, 64, 900, 833, 64, False),
                                                          (1, 16, 128, 1025, 1025, 0, False), (2, 8, 64, 1000, 700, 100, True)])
def test_blocks_dealt_to_the_cus(gu, B, H, D, P, v, vis_start, with_pos):
    """More than one workgroup per CU and one round of them: blocks come in another order than by their length, over several sequences."""
    q = di.normal((B, P, H, D), "bf16", 1101 + P, di.STREAM_PREFILL_Q)
    k = di.normal((B, H, P + 3, D), "bf16", 1102 + P, di.STREAM_K)
    pos = np.stack([np.random.default_rng(P + b).permutation(P) for b in range(B)]).astype(np.int32) if with_pos else None
    scores, _, _ = gu.run_compress("bf16", q, k, P, vis_start, v, 1, 2, q_pos=pos)
    np.testing.assert_allclose(scores, oracle.visual_scores(q, k, "bf16", vis_start, v, q_pos=pos), rtol=SCORE_RTOL["bf16"])


# sizes, and whether workgroups of 128 keys or rows take the column sums with given log-sum-exps, those without, and the log-sum-exps (tests/test_score_plan.py asks the plan)
TWO_BLOCKS = [((32, 32, 32, 64, 200, 129, 3), (1, 1, 0)), ((32, 32, 8, 64, 321, 250, 0), (1, 1, 0)), ((15, 32, 32, 128, 520, 300, 17), (1, 1, 1)), ((18, 32, 8, 128, 449, 385, 64), (1, 1, 1)),
              ((16, 32, 8, 128, 600, 340, 5), (1, 1, 1)), ((27, 16, 8, 256, 300, 200, 0), (1, 1, 1)), ((27, 16, 16, 256, 330, 193, 70), (1, 1, 1)), ((27, 16, 8, 256, 400, 300, 9), (1, 1, 1))]


@pytest.mark.parametrize("with_pos", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,D,P,v,vis_start", [sizes for sizes, _ in TWO_BLOCKS])
def test_workgroups_of_two_blocks(gu, B, Hq, Hkv, D, P, v, vis_start, with_pos):
    """Enough sequences for workgroups of 128 keys or rows, at odd and even numbers of 64s, against the same tensors one element further on, which take blocks of 64.
    Column sums add the same terms in the same order: the same bits where the log-sum-exps are given.  Those themselves and the entropies are float32 sums of
    a few hundred positive terms in another order: 2e-5 of a score, and of an entropy's scale (logarithms up to 10)."""
    import torch
    import paper_2505_19201_amd as dream
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1701 + P)
    q = torch.empty(B, P, Hq, D, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    k = torch.empty(B, Hkv, P + 1, D, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    lse = torch.rand(B, Hq, P, generator=gen, device="cuda") + 5.0
    pos = torch.stack([torch.randperm(P, generator=gen, device="cuda") for _ in range(B)]).int() if with_pos else None
    desc = dream.attn_desc(B, Hq, Hkv, D, dream.BF16, P + 1)

    def results(q, k):
        out = []
        for given in (lse, None):
            scores = torch.full((B, v), float("nan"), device="cuda")
            dream.dream_visual_compress(desc, q, pos, P, k, P, vis_start, v, 0, 1, None, scores, None, None, 0, None, 0,
                                        gu.workspace(dream.dream_visual_compress_workspace(desc, P, v)), row_lse_in=given)
            out.append(scores)
        row, ae = torch.full((B, Hq, P), float("nan"), device="cuda"), torch.full((B,), float("nan"), device="cuda")
        dream.dream_attention_entropy(desc, q, pos, P, k, P, row, ae, gu.workspace(dream.dream_attention_entropy_workspace(desc, P)))
        return [x.cpu().numpy() for x in (*out, row, ae)]

    q1 = torch.empty(q.numel() + 1, dtype=q.dtype, device="cuda")[1:].view(q.shape).copy_(q)
    assert q1.data_ptr() % 16 == 2
    got, want = results(q, k), results(q1, k)
    assert all(np.isfinite(x).all() for x in got)
    assert np.array_equal(got[0], want[0])
    np.testing.assert_allclose(got[1], want[1], rtol=2e-5)
    np.testing.assert_allclose(got[2], want[2], rtol=0, atol=2e-4 / 10)
    np.testing.assert_allclose(got[3], want[3], rtol=0, atol=2e-4 / 10)


@pytest.mark.parametrize("D,P,v", [(128, 1279, 1023), (64, 333, 300), (256, 449, 200)])
def test_stale_workspace_is_never_read(gu, D, P, v):
    """Blocks with fewer splits than others, in both score passes, over a workspace of NaN patterns (the harness fills it)."""
    q = di.normal((1, P, 4, D), "bf16", 1101 + P, di.STREAM_PREFILL_Q)
    k = di.normal((1, 2, P, D), "bf16", 1102 + P, di.STREAM_K)
    scores, _, _ = gu.run_compress("bf16", q, k, P, 0, v, 1, 2)
    np.testing.assert_allclose(scores, oracle.visual_scores(q, k, "bf16", 0, v), rtol=SCORE_RTOL["bf16"])


@pytest.mark.parametrize("v", [40, 576, 1500, 2500])
@pytest.mark.parametrize("num,den", [(1, 2), (3, 4), (1, 1)])
def test_every_score_is_a_token_even_the_lowest_key(gu, v, num, den):
    """Scores that are NaN patterns of all ones, the lowest of all keys: exactly k distinct tokens are kept, lower ones first among
    equals, and the gather follows them.  (Host scores in sort order: larger key first, the key being the float's bits made monotone.)"""
    g = di.rng(19 + v, di.STREAM_SCORES)
    s = g.standard_normal(size=(2, v)).astype(np.float32)
    s.view(np.uint32)[0, g.permutation(v)[: (v * 3) // 5]] = 0xFFFFFFFF
    s.view(np.uint32)[1] = 0xFFFFFFFF
    rows = di.normal((2, v + 3, 8), "bf16", 1200 + v, di.STREAM_ROWS)
    _, kept, gathered = gu.run_compress("bf16", None, None, 0, 3, v, num, den, scores_in=s, gather_src=rows)
    u = s.view(np.uint32).astype(np.int64)
    key = np.where(u & 0x80000000, 0xFFFFFFFF - u, u | 0x80000000)
    k = oracle.keep_count(v, num, den)
    want = np.sort(np.argsort(-key, axis=1, kind="stable")[:, :k], axis=1) + 3
    assert np.array_equal(kept, want)
    assert np.array_equal(gathered, oracle.gather_rows(rows, "bf16", want.astype(np.int32)))


@pytest.mark.parametrize("D,P,v", [(64, 333, 300), (128, 200, 129), (256, 97, 64)])
@pytest.mark.parametrize("shift_q,shift_k", [(1, 0), (0, 3), (4, 4)])
def test_rows_that_are_not_16_byte_aligned(gu, D, P, v, shift_q, shift_k):
    """q and the cache as slices that start a few elements into a larger buffer: the loads straight to LDS need 16-byte alignment, so these
    calls take another way, with the same bits in every result (both score passes, positions, the entropy)."""
    import torch
    import paper_2505_19201_amd as dream
    q = di.normal((2, P, 4, D), "bf16", 1301 + P, di.STREAM_PREFILL_Q)
    k = di.normal((2, 2, P + 1, D), "bf16", 1302 + P, di.STREAM_K)
    pos = dream.to_device(np.stack([di.rng(1303 + P, di.STREAM_SCORES).permutation(P) for _ in range(2)]).astype(np.int32))
    desc = dream.attn_desc(2, 4, 2, D, dream.BF16, P + 1)

    def placed(a, shift):
        flat = torch.zeros(a.size + 16, dtype=torch.bfloat16, device="cuda")
        t = flat[shift:shift + a.size].view(a.shape)
        assert t.data_ptr() % 16 == shift * 2 and t.is_contiguous()
        return t.copy_(dream.to_device(a, "bf16"))

    def results(sq, sk):
        dq, dk = placed(q, sq), placed(k, sk)
        out = []
        for p in (None, pos):
            scores = torch.full((2, v), float("nan"), device="cuda")
            kept = torch.full((2, oracle.keep_count(v, 1, 2)), -7, dtype=torch.int32, device="cuda")
            dream.dream_visual_compress(desc, dq, p, P, dk, P, 0, v, 1, 2, None, scores, kept, None, 0, None, 0,
                                        gu.workspace(dream.dream_visual_compress_workspace(desc, P, v)))
            row = torch.full((2, 4, P), float("nan"), device="cuda")
            ae = torch.full((2,), float("nan"), device="cuda")
            dream.dream_attention_entropy(desc, dq, p, P, dk, P, row, ae, gu.workspace(dream.dream_attention_entropy_workspace(desc, P)))
            out += [scores, kept, row, ae]
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out]

    for got, want in zip(results(shift_q, shift_k), results(0, 0)):
        assert np.isfinite(got).all() and np.array_equal(got, want)


@pytest.mark.parametrize("v", [1, 255, 256, 257, 768, 769, 1281, 1793])
@pytest.mark.parametrize("B,row_elems", [(1, 8), (2, 1000), (1, 8200), (40, 64), (3, 7)])
def test_selection_with_its_rows(gu, v, B, row_elems):
    """Registers filled to the last token and one over; rows copied by the selection's own workgroups (few sequences) and by a launch of
    their own (40 sequences), rows of fewer chunks than lanes, of more, and of bytes that are no multiple of 16.  Scores with ties: bit for bit."""
    rng = np.random.default_rng(v * 31 + B)
    scores = rng.integers(0, max(v // 3, 2), size=(B, v)).astype(np.float32) / 7.0
    src = rng.integers(0, 1 << 16, size=(B, v + 5, row_elems)).astype(np.uint16)
    _, kept, rows = gu.run_compress("bf16", None, None, v + 5, 3, v, 1, 2, scores_in=scores, gather_src=src)
    want = oracle.topk_keep(scores, 3, 1, 2)
    assert np.array_equal(kept, want)
    for b in range(B):
        assert np.array_equal(rows[b], src[b][want[b]])


@pytest.mark.parametrize("v", [1, 64, 65, 257, 600, 1088, 2047, 2048])
@pytest.mark.parametrize("bit", [-1, 0, 3, 4, 11, 15, 20, 28, 31])
def test_selection_from_the_first_bit_that_differs(gu, v, bit):
    """Scores that agree in all bits above `bit` (-1: in all), kept shares from one token to all of them, ties at the cut."""
    g = di.rng(91, 905, v * 64 + bit + 1)
    low = g.integers(0, 1 << (bit + 1), size=v, dtype=np.int64) if bit >= 0 else np.zeros(v, dtype=np.int64)
    low[::3] = low[0]
    s = ((0x3f5a5a5a5a & ~((1 << (bit + 1)) - 1) | low) & 0xffffffff).astype(np.uint32).view(np.float32)[None]
    s = np.nan_to_num(s, nan=0.5, posinf=3.0e38, neginf=-3.0e38)
    for num, den in ((1, v), (1, 4), (2, 3), (1, 1)):
        _, kept, _ = gu.run_compress("bf16", None, None, 0, 3, v, num, den, scores_in=s)
        assert np.array_equal(kept, oracle.topk_keep(s.astype(np.float64), 3, num, den)), (num, den)
