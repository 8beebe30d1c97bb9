"""GPU parity: dream_attention_entropy (Eq. 2) against the float64 oracle.

Tolerance: the entropy is LSE minus the attention-weighted mean score, two float32 sums over up to ~1600 keys of
exact bf16 products, values of order 1..10: |error| <= 2e-4 (bf16 tensors), 2e-5 (float32 tensors)."""
import numpy as np
import pytest

import dream_inputs as di
import oracle

pytestmark = pytest.mark.gpu
TOL = {"f32": 2e-5, "bf16": 2e-4}


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from tests import gpu_util
    return gpu_util


def _check(gu, cfg, n_q=None, q_pos=None, scale=None):
    q = di.prefill_q(cfg, n_q=n_q)
    k = di.verify_inputs(cfg).k
    n_keys = cfg.prefix
    row, ae = gu.run_entropy(cfg.dtype, q, k, n_keys, q_pos=q_pos, scale=0.0 if scale is None else scale)
    want_row, want_ae = oracle.attention_entropy(q, k, cfg.dtype, q_pos=q_pos, scale=scale)
    assert np.isfinite(row).all()
    assert np.abs(row - want_row).max() <= TOL[cfg.dtype], np.abs(row - want_row).max()
    assert np.abs(ae - want_ae).max() <= TOL[cfg.dtype]
    return row, ae


def test_tiny_f32(gu):
    _check(gu, di.CONFIGS["tiny"])


@pytest.mark.parametrize("Hq,Hkv,D,n", [(4, 4, 64, 200), (8, 2, 128, 333), (4, 2, 256, 97), (2, 1, 64, 1), (4, 4, 128, 65)])
def test_small_bf16_shapes_span_tiles_and_ragged_tails(gu, Hq, Hkv, D, n):
    cfg = di.Config("e", "bf16", 2, Hq, Hkv, D, Hq * D, n, 0, 4, 2, 1, 2, 100, 1, 31)
    _check(gu, cfg)


def test_explicit_positions_and_scale(gu):
    cfg = di.Config("e", "bf16", 2, 4, 2, 128, 512, 150, 0, 4, 2, 1, 2, 100, 1, 32)
    pos = np.stack([di.rng(5, 500, b).integers(0, 150, size=40) for b in range(2)]).astype(np.int32)
    _check(gu, cfg, n_q=40, q_pos=pos, scale=0.31)
    cfg32 = di.Config("e", "f32", 1, 4, 4, 64, 256, 90, 0, 4, 2, 1, 2, 100, 1, 33)
    _check(gu, cfg32, n_q=17, q_pos=np.arange(17, dtype=np.int32)[None] * 5)


def test_zero_queries_reproduce_log_count(gu):
    cfg = di.Config("e", "bf16", 1, 4, 4, 128, 512, 300, 0, 4, 2, 1, 2, 100, 1, 34)
    q = np.zeros_like(di.prefill_q(cfg))
    k = di.verify_inputs(cfg).k
    row, ae = gu.run_entropy("bf16", q, k, 300)
    np.testing.assert_allclose(row, np.broadcast_to(np.log(np.arange(1, 301)), row.shape), atol=TOL["bf16"])


@pytest.mark.parametrize("name", ["llava", "pixtral", "gemma3", "smolvlm_b8"])
def test_full_size_configs(gu, name):
    cfg = di.CONFIGS[name]
    _check(gu, cfg)


# whole blocks and split ones, in the order of the blocks or dealt to the CUs, with heads that divide 256 and others, one sequence and several
@pytest.mark.parametrize("B,Hq,Hkv,D,n,with_pos", [(2, 16, 16, 64, 700, False), (2, 8, 2, 64, 1279, False), (3, 7, 7, 64, 900, False), (1, 16, 4, 128, 1025, False),
                                                   (2, 8, 8, 64, 1000, True), (5, 1, 1, 64, 1600, False), (1, 32, 8, 64, 1601, False),
                                                   (2, 40, 8, 64, 1700, False)])      # (the last: more sums than the mean asks for at once)
def test_blocks_whole_and_split(gu, B, Hq, Hkv, D, n, with_pos):
    cfg = di.Config("e", "bf16", B, Hq, Hkv, D, Hq * D, n, 0, 4, 2, 1, 2, 100, 1, 38)
    pos = np.stack([np.random.default_rng(39 + b).permutation(n) for b in range(B)]).astype(np.int32) if with_pos else None
    _check(gu, cfg, q_pos=pos)


@pytest.mark.parametrize("B,Hq,Hkv,D,n", [(1, 4, 4, 128, 1279), (2, 8, 2, 64, 333), (1, 2, 1, 256, 449)])
def test_stale_workspace_is_never_read(gu, B, Hq, Hkv, D, n):
    """Row blocks of the causal triangle have different numbers of key splits; what a block leaves out counts as nothing,
    whatever the workspace held before (the harness fills it with 0xFF bytes, NaN as floats)."""
    cfg = di.Config("e", "bf16", B, Hq, Hkv, D, Hq * D, n, 0, 4, 2, 1, 2, 100, 1, 35)
    row, ae = _check(gu, cfg)
    assert (row[:, :, 1:] > 0).all() and (ae > 0).all()      # only the first row sees a single key


@pytest.mark.parametrize("dtype,Hq,Hkv,D,n", [("bf16", 4, 4, 64, 200), ("bf16", 8, 2, 128, 333), ("bf16", 2, 1, 256, 449), ("bf16", 2, 2, 128, 1279), ("f32", 4, 2, 64, 90)])
def test_a_nan_score_reaches_the_rows_that_see_it(gu, dtype, Hq, Hkv, D, n):
    """One key of NaN scores, at the edges of the steps and of the key splits: exactly the rows that see it become NaN, whether the key lies in
    a step with masked keys (the rows' diagonal, the ragged end, explicit positions) or in one without; the others keep every bit.  A row of
    NaN scores alone is NaN too."""
    cfg = di.Config("e", dtype, 1, Hq, Hkv, D, Hq * D, n, 0, 4, 2, 1, 2, 100, 1, 36)
    q, k = di.prefill_q(cfg), di.verify_inputs(cfg).k
    nan = np.float32(np.nan) if dtype == "f32" else np.uint16(0x7FC0)
    pos = np.stack([np.random.default_rng(37).permutation(n)]).astype(np.int32)
    for q_pos in (None, pos):
        at = np.arange(n) if q_pos is None else q_pos[0]
        base, _ = gu.run_entropy(dtype, q, k, n, q_pos=q_pos)
        assert np.isfinite(base).all()
        for key in sorted({0, 1, 31, 63, 64, n // 2, n - 1}):
            kn = k.copy()
            kn[0, Hkv - 1, key, D // 2] = nan
            row, ae = gu.run_entropy(dtype, q, kn, n, q_pos=q_pos)
            want, _ = oracle.attention_entropy(q, kn, dtype, q_pos=q_pos) if n < 100 else (None, None)
            hit = np.zeros(base.shape, dtype=bool)
            hit[0, Hq - Hq // Hkv:] = at >= key
            assert np.array_equal(np.isnan(row), hit), (key, np.isnan(row).sum(), hit.sum())
            assert want is None or np.array_equal(np.isnan(want), hit)
            assert np.array_equal(row[~hit], base[~hit])
            assert np.isnan(ae).all() == hit.any()
        qn = q.copy()
        rows = sorted({0, 1, n // 3, n - 1})
        qn[0, rows, 0, 0] = nan
        row, ae = gu.run_entropy(dtype, qn, k, n, q_pos=q_pos)
        hit = np.zeros(base.shape, dtype=bool)
        hit[0, 0, rows] = True
        assert np.array_equal(np.isnan(row), hit) and np.array_equal(row[~hit], base[~hit]) and np.isnan(ae).all()
