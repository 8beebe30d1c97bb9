"""GPU parity: dream_project_rows (the linear maps of Eq. 1) against the float64 oracle.

Tolerance: the products of bf16 values are exact in float32 and the MFMA accumulates in float32, so the error is
the bf16 rounding of the stored result: |err| <= 2^-8 |y| + 1e-3.  Cache rows that the call does not address
must keep their bytes."""
import numpy as np
import pytest

import dream_inputs as di
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from tests import gpu_util
    return gpu_util


def _inputs(B, R, hidden, H, D, seed):
    x = di.normal((B, R, hidden), "bf16", seed, di.STREAM_ROWS)
    w32 = di.normal((H * D, hidden), "f32", seed + 1, di.STREAM_ROWS) * np.float32(1.0 / np.sqrt(hidden))
    return x, di.f32_to_bf16_bits(w32)


def _close(got, want):
    err = np.abs(got - want)
    assert (err <= np.abs(want) / 256 + 1e-3).all(), err.max()


@pytest.mark.parametrize("B,R,hidden,H,D", [(1, 1, 4096, 32, 128), (1, 10, 4096, 32, 128), (1, 60, 4096, 32, 128), (2, 7, 5120, 8, 128),
                                            (1, 16, 3840, 16, 256), (8, 10, 2048, 32, 64), (3, 33, 256, 2, 16), (30, 11, 512, 4, 64)])
def test_dense_queries(gu, B, R, hidden, H, D):
    x, w = _inputs(B, R, hidden, H, D, 40 + R)
    got = gu.run_project(x, w, H, D)
    _close(got, oracle.project(x, w, "bf16", H, D))


@pytest.mark.parametrize("B,R,hidden,H,D,with_index", [(1, 7, 4096, 32, 128, False), (2, 10, 4096, 8, 128, True), (4, 20, 2048, 32, 64, True)])
def test_cache_append(gu, B, R, hidden, H, D, with_index):
    x, w = _inputs(B, R, hidden, H, D, 60 + R)
    s_max, T = 150, 40
    cache = di.normal((B, H, s_max, D), "bf16", 77, di.STREAM_K)
    row_base = np.array([90 - 7 * b for b in range(B)], dtype=np.int32)
    g = di.rng(78, 800)
    row_index = np.stack([np.sort(g.choice(T, size=R, replace=False)) for _ in range(B)]).astype(np.int32) if with_index else None
    got = gu.run_project(x, w, H, D, row_base=row_base, row_index=row_index, cache=cache)
    want = oracle.project(x, w, "bf16", H, D)
    touched = np.zeros((B, s_max), dtype=bool)
    for b in range(B):
        for r in range(R):
            row = int(row_base[b]) + (int(row_index[b, r]) if with_index else r)
            touched[b, row] = True
            vals = di.bf16_bits_to_f32(got[b, :, row].view(np.uint16)).astype(np.float64)      # [H, D]
            _close(vals, want[b, r])
    keep = ~touched
    for b in range(B):
        assert np.array_equal(got[b][:, keep[b]], cache[b][:, keep[b]].view(np.int16))         # every other row untouched


def test_identity_weight_copies_rows_exactly(gu):
    hidden = 256
    x = di.normal((2, 5, hidden), "bf16", 91, di.STREAM_ROWS)
    w = di.f32_to_bf16_bits(np.eye(hidden, dtype=np.float32))
    got = gu.run_project(x, w, 4, 64)
    assert np.array_equal(got.reshape(2, 5, hidden), di.as_f64(x, "bf16"))


@pytest.mark.parametrize("B,R,hidden,Hq,Hkv,D", [(1, 10, 5120, 32, 8, 128), (3, 10, 2048, 32, 32, 64), (2, 20, 3840, 16, 8, 256)])
def test_one_launch_for_a_draft_level(gu, B, R, hidden, Hq, Hkv, D):
    e = di.normal((B, R, hidden), "bf16", 101, di.STREAM_ROWS)
    s = di.normal((B, R, hidden), "bf16", 102, di.STREAM_ROWS)
    ws = [di.f32_to_bf16_bits(di.normal((h * D, hidden), "f32", 103 + i, di.STREAM_ROWS) * np.float32(hidden ** -0.5))
          for i, h in enumerate((Hq, Hkv, Hkv))]
    s_max = 120
    kc = di.normal((B, Hkv, s_max, D), "bf16", 110, di.STREAM_K)
    vc = di.normal((B, Hkv, s_max, D), "bf16", 111, di.STREAM_V)
    row_base = np.array([70 - 5 * b for b in range(B)], dtype=np.int32)
    g = di.rng(112, 800)
    row_index = np.stack([np.sort(g.choice(40, size=R, replace=False)) for _ in range(B)]).astype(np.int32)
    q, k, v = gu.run_project_qkv(e, s, ws[0], ws[1], ws[2], Hq, Hkv, D, row_base, row_index, kc, vc)
    _close(q, oracle.project(e, ws[0], "bf16", Hq, D))
    for got, w, cache in ((k, ws[1], kc), (v, ws[2], vc)):
        want = oracle.project(s, w, "bf16", Hkv, D)
        for b in range(B):
            rows = row_base[b] + row_index[b]
            _close(di.bf16_bits_to_f32(got[b][:, rows].view(np.uint16)).astype(np.float64), want[b].transpose(1, 0, 2))
            keep = np.ones(s_max, dtype=bool)
            keep[rows] = False
            assert np.array_equal(got[b][:, keep], cache[b][:, keep].view(np.int16))


def test_rows_outside_the_cache_are_dropped(gu):
    B, R, hidden, H, D, s_max = 1, 6, 256, 2, 64, 20
    x, w = _inputs(B, R, hidden, H, D, 120)
    cache = di.normal((B, H, s_max, D), "bf16", 121, di.STREAM_K)
    row_index = np.array([[0, 1, 2, 3, 4, -40]], dtype=np.int32)          # base 16: rows 16..19, then 20 (out) and -24 (out)
    got = gu.run_project(x, w, H, D, row_base=np.array([16], dtype=np.int32), row_index=row_index, cache=cache)
    want = oracle.project(x, w, "bf16", H, D)
    assert np.array_equal(got[0][:, :16], cache[0][:, :16].view(np.int16))
    for r in range(4):
        _close(di.bf16_bits_to_f32(got[0][:, 16 + r].view(np.uint16)).astype(np.float64), want[0, r])


@pytest.mark.parametrize("R", [17, 40, 56, 65, 96, 97, 128, 129, 260])
@pytest.mark.parametrize("hidden,tiles", [(256, 300), (768, 700), (1280, 64)])
def test_tiles_of_a_workgroup(gu, R, hidden, tiles):
    """Every number of row tiles with one, two and three feature tiles (two at most beside seven and eight row tiles), waves with no, one and
    several steps of the hidden dimension, a last workgroup with fewer feature tiles and a last pass with fewer rows."""
    x, w = _inputs(1, R, hidden, tiles, 16, 140 + R)
    _close(gu.run_project(x, w, tiles, 16), oracle.project(x, w, "bf16", tiles, 16))


@pytest.mark.parametrize("B,R,hidden,H,D", [(1, 17, 512, 5, 16), (1, 32, 256, 5, 16), (3, 11, 768, 1, 48), (1, 65, 256, 3, 32), (7, 14, 512, 3, 16),
                                            (1, 113, 256, 4, 16), (1, 128, 256, 4, 16), (1, 129, 256, 4, 16), (1, 20, 256, 770, 16)])
def test_row_and_feature_tile_edges(gu, B, R, hidden, H, D):
    """One row past a tile, whole tiles, every tile count, a second pass (129 rows), a last workgroup with fewer feature tiles (770)."""
    x, w = _inputs(B, R, hidden, H, D, 140 + R)
    _close(gu.run_project(x, w, H, D), oracle.project(x, w, "bf16", H, D))


@pytest.mark.parametrize("R", [129, 150, 200, 321, 513])
@pytest.mark.parametrize("hidden,Hq,Hkv,D", [(256, 5, 3, 16), (768, 12, 12, 64), (1280, 70, 9, 32)])
def test_passes_side_by_side(gu, R, hidden, Hq, Hkv, D):
    """More than 128 rows: several workgroups share a feature tile's rows (or one goes through them), three maps of different widths, a number of feature tiles that
    is no multiple of 8, a last pass with one row or several."""
    e = di.normal((1, R, hidden), "bf16", 301, di.STREAM_ROWS)
    s = di.normal((1, R, hidden), "bf16", 302, di.STREAM_ROWS)
    ws = [di.f32_to_bf16_bits(di.normal((h * D, hidden), "f32", 303 + i, di.STREAM_ROWS) * np.float32(hidden ** -0.5))
          for i, h in enumerate((Hq, Hkv, Hkv))]
    kc = di.normal((1, Hkv, R + 9, D), "bf16", 310, di.STREAM_K)
    vc = di.normal((1, Hkv, R + 9, D), "bf16", 311, di.STREAM_V)
    row_index = np.arange(R, dtype=np.int32)[None]
    q, k, v = gu.run_project_qkv(e, s, ws[0], ws[1], ws[2], Hq, Hkv, D, np.array([4], dtype=np.int32), row_index, kc, vc)
    _close(q, oracle.project(e, ws[0], "bf16", Hq, D))
    for got, w, cache in ((k, ws[1], kc), (v, ws[2], vc)):
        _close(di.bf16_bits_to_f32(got[0][:, 4:4 + R].view(np.uint16)).astype(np.float64), oracle.project(s, w, "bf16", Hkv, D)[0].transpose(1, 0, 2))
        assert np.array_equal(got[0][:, :4], cache[0][:, :4].view(np.int16)) and np.array_equal(got[0][:, 4 + R:], cache[0][:, 4 + R:].view(np.int16))


@pytest.mark.parametrize("R", [1, 4, 5, 8, 9, 12, 13, 16])
@pytest.mark.parametrize("hidden,tiles", [(256, 1), (768, 256), (1280, 257), (768, 511), (768, 513), (4096, 258), (2048, 257), (2304, 511), (2304, 513), (1792, 300)])
def test_up_to_sixteen_rows(gu, R, hidden, tiles):
    """Both kernels on both sides of the lines between them (256 and 512 feature tiles, 8 rows, a hidden dimension of 2048, rows a multiple of 8 KB apart), one to four pieces of rows, a
    workgroup with one tile of two, a wave whose share of the hidden dimension ends in half a step."""
    x, w = _inputs(1, R, hidden, tiles, 16, 150 + R)
    _close(gu.run_project(x, w, tiles, 16), oracle.project(x, w, "bf16", tiles, 16))


@pytest.mark.parametrize("hidden,Hq,Hkv", [(512, 7, 3), (512, 151, 55), (512, 255, 129), (512, 171, 171), (2048, 151, 55), (2048, 255, 129), (2048, 171, 171)])
def test_maps_of_odd_widths_in_one_launch(gu, hidden, Hq, Hkv):
    """Every map's last workgroup has one feature tile of two, and none writes into another map."""
    B, R, D = 1, 10, 16
    e, s = (di.normal((B, R, hidden), "bf16", 401 + i, di.STREAM_ROWS) for i in range(2))
    ws = [di.f32_to_bf16_bits(di.normal((h * D, hidden), "f32", 403 + i, di.STREAM_ROWS) * np.float32(hidden ** -0.5)) for i, h in enumerate((Hq, Hkv, Hkv))]
    kc, vc = (di.normal((B, Hkv, 40, D), "bf16", 410 + i, di.STREAM_K) for i in range(2))
    row_index = np.array([[9, 0, 3, 1, 30, 12, 5, 6, 7, 35]], dtype=np.int32)              # 35: outside the cache
    q, k, v = gu.run_project_qkv(e, s, ws[0], ws[1], ws[2], Hq, Hkv, D, np.array([5], dtype=np.int32), row_index, kc, vc)
    _close(q, oracle.project(e, ws[0], "bf16", Hq, D))
    for got, w, cache in ((k, ws[1], kc), (v, ws[2], vc)):
        want = oracle.project(s, w, "bf16", Hkv, D)[0].transpose(1, 0, 2)
        rows = 5 + row_index[0, :9]
        _close(di.bf16_bits_to_f32(got[0][:, rows].view(np.uint16)).astype(np.float64), want[:, :9])
        keep = np.ones(40, dtype=bool)
        keep[rows] = False
        assert np.array_equal(got[0][:, keep], cache[0][:, keep].view(np.int16))


@pytest.mark.parametrize("hidden,R,tiles", [(512, 8, (31, 17, 5, 9)), (512, 2, (99, 101, 55, 77)), (512, 8, (299, 101, 85, 77)), (2048, 5, (99, 101, 55, 77)), (256, 10, (99, 1, 55, 77)),
                                            (256, 10, (199, 188, 170, 181)), (256, 130, (199, 188, 170, 181))])
def test_four_maps_in_one_launch(gu, hidden, R, tiles):
    """As many maps as a call takes, dense and into caches in turn, some rows outside the cache: one feature tile a workgroup, the small workgroups, two tiles and three, where the last
    workgroup of a map lacks one or two; several passes over the rows."""
    import torch
    import paper_2505_19201_amd as dream
    B, D, s_max = 2, 16, 300
    xs = [di.normal((B, R, hidden), "bf16", 501 + i, di.STREAM_ROWS) for i in range(4)]
    ws = [di.f32_to_bf16_bits(di.normal((t * D, hidden), "f32", 511 + i, di.STREAM_ROWS) * np.float32(hidden ** -0.5)) for i, t in enumerate(tiles)]
    base = np.array([7, 160], dtype=np.int32)
    index = np.stack([di.rng(520 + b, 800).permutation(s_max)[:R] for b in range(B)]).astype(np.int32)    # (some past the end, behind the base)
    place = [None, base[:, None] + np.arange(R)[None], None, base[:, None] + index]
    rb, ri = dream.to_device(base), dream.to_device(index)
    fill = 1024.0             # (results are about 1: no row that was written holds it)
    outs = [torch.full((B, R, t, D) if i % 2 == 0 else (B, t, s_max, D), fill, dtype=torch.bfloat16, device="cuda") for i, t in enumerate(tiles)]
    jobs = [(dream.to_device(xs[i], "bf16"), dream.to_device(ws[i], "bf16"), t, rb if i % 2 else None, ri if i == 3 else None, outs[i]) for i, t in enumerate(tiles)]
    dream.dream_project_rows_multi(dream.attn_desc(B, 1, 1, D, dream.BF16, s_max), jobs, R, hidden)
    torch.cuda.synchronize()
    for i, t in enumerate(tiles):
        want = oracle.project(xs[i], ws[i], "bf16", t, D)
        got = gu.out_to_f64(outs[i])
        if i % 2 == 0:
            _close(got, want)
            continue
        full = np.full(got.shape, fill)
        for b in range(B):
            for r in range(R):
                if 0 <= place[i][b, r] < s_max:
                    full[b, :, place[i][b, r]] = want[b, r]
        _close(got, full)
        assert np.array_equal(got == fill, full == fill)
