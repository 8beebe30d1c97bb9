"""GPU parity: dream_accept_path against the oracle, bit-exact on every integer output."""
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


def _compare(gu, logits, dtype, token, parent, max_depth):
    got = gu.run_accept(logits, dtype, token, parent, max_depth)
    want = oracle.accept_path(logits, dtype, token, parent, max_depth)
    for g, w, what in zip(got, want, ("node_argmax", "accept_len", "accept_path", "bonus_token")):
        assert np.array_equal(g, w), what
    return got


def test_tiny_config_every_plant_depth(gu):
    cfg = di.CONFIGS["tiny"]
    for d in range(cfg.depth + 1):
        logits, token, parent, ends = di.accept_inputs(cfg, plant_depths=[d])
        got = _compare(gu, logits, cfg.dtype, token, parent, cfg.depth)
        assert got[1][0] == d


@pytest.mark.parametrize("name", ["llava", "pixtral", "gemma3", "smolvlm_b8", "smolvlm_b32"])
def test_full_size_configs(gu, name):
    cfg = di.CONFIGS[name]
    logits, token, parent, ends = di.accept_inputs(cfg, n_ties=2)
    got = _compare(gu, logits, cfg.dtype, token, parent, cfg.depth)
    assert got[1].tolist() == [b % (cfg.depth + 1) for b in range(cfg.batch)]
    assert (got[1] + 1 <= 7).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("vocab", [1, 7, 1000, 8191, 8192, 8193, 32003])
def test_ragged_vocab_and_planted_ties(gu, dtype, vocab):
    T = 13
    parent = di.random_tree(T, 4, 5 + vocab)
    token = di.tree_tokens(parent, max(vocab, T), 6)[None] % vocab
    logits = di.normal((2, T, vocab), dtype, 70 + vocab, di.STREAM_LOGITS)
    top = np.float32(9.0) if dtype == "f32" else di.f32_to_bf16_bits(np.array([9.0], dtype=np.float32))[0]
    g = di.rng(3, 902, vocab)
    for b in range(2):
        for i in range(T):
            cols = g.integers(0, vocab, size=3)
            logits[b, i, cols] = top                      # exact ties at the maximum, anywhere in the row
    _compare(gu, logits, dtype, np.repeat(token, 2, 0), np.repeat(parent[None], 2, 0), 4)


def _argmax(x):
    """First index of the largest value, NaN passed over; a row without anything above -inf: not compared."""
    return np.argmax(np.where(np.isnan(x), -np.inf, x), axis=-1)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,vocab,depth", [(1, 9, 3), (2, 8, 0), (63, 4096, 5), (64, 16392, 2), (64, 8200, 70), (65, 8200, 70), (64, 50003, 4), (65, 16384, 2), (600, 40, 9),
                                           (7, 1024, 3), (7, 1031, 3), (7, 2048, 3), (7, 2063, 3), (7, 4097, 3), (7, 4111, 3)])      # (around one piece a thread, and half of them)
def test_masked_logits_and_both_walks(gu, dtype, T, vocab, depth):
    """Trees on both sides of 64 nodes, chains deeper than a wave, depth limits; logits of which most are -inf, some NaN (quiet and signalling), zeros of both signs, and ties in the
    same 16 bytes, the same thread and others; rows on and off the 16-byte boundaries, chunks without and with a tail."""
    g = di.rng(41, 903, vocab + T)
    chain = depth >= 64
    parent = np.array([[i - 1 for i in range(T)]] * 3 if chain else [di.random_tree(T, 5, 42 + b) if T > 1 else [-1] for b in range(3)], dtype=np.int32)
    x = g.normal(size=(3, T, vocab)).astype(np.float32)
    x = np.where(g.uniform(size=x.shape) < 0.7, np.float32(-np.inf), x)
    x[..., g.integers(0, vocab, size=3)] = 0.0
    x[0] = np.where(x[0] > 0, np.float32(-0.0), x[0])                 # zeros are the maximum of the first sequence, of either sign
    x[0, :, vocab // 2] = 0.0
    x[1, :, vocab // 3] = x[1, :, min(vocab // 3 + 1, vocab - 1)] = x[1, :, vocab - 1] = 7.0
    x[2, :, vocab - 1] = 8.0
    bits = di.f32_to_bf16_bits(x) if dtype == "bf16" else x.view(np.uint32).copy()
    quiet, signalling = (0x7fc1, 0x7f81) if dtype == "bf16" else (0x7fc00001, 0x7f800001)
    for nan in (quiet, signalling):
        where = g.uniform(size=bits.shape) < 0.05
        where[..., [vocab // 2, vocab // 3, vocab - 1]] = False
        bits[where] = nan
    logits = bits if dtype == "bf16" else bits.view(np.float32)
    am = _argmax(di.bf16_bits_to_f32(bits) if dtype == "bf16" else logits).astype(np.int32)
    token = g.integers(0, vocab, size=(3, T)).astype(np.int32)
    follow = g.uniform(size=(3, T)) < (0.98 if chain else 0.6)         # these tokens are their parents' arg-max
    for b in range(3):
        for i in range(1, T):
            if follow[b, i]:
                token[b, i] = am[b, parent[b, i]]
    node_argmax, accept_len, path, bonus = gu.run_accept(logits, dtype, token, parent, depth)
    assert np.array_equal(node_argmax, am)
    for b in range(3):
        d = [0] + [-1] * (T - 1)
        for i in range(1, T):
            p = parent[b, i]
            if d[p] >= 0 and token[b, i] == am[b, p] and d[p] < depth:
                d[i] = d[p] + 1
        end = int(np.argmax(d))
        want, n = [-1] * (depth + 1), end
        for t in range(d[end], -1, -1):
            want[t], n = n, parent[b, n]
        assert accept_len[b] == d[end] and path[b].tolist() == want and bonus[b] == am[b, end]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V", [1, 3, 9, 300, 8192, 8200, 16384, 16387, 50257])
def test_rows_without_anything_above_minus_infinity(gu, dtype, V):
    """Fully masked rows (all -inf; -inf and NaN; all NaN) have index 0 as the oracle has, on and off the 16-byte boundaries, over one chunk and several, with and without a tail; a
    chunk of -inf does not take the row from a finite logit in another one."""
    import torch
    import paper_2505_19201_amd as dream
    x = np.full((1, 6, V), -np.inf, dtype=np.float32)
    x[0, 1, V // 2] = np.nan
    x[0, 2, 1:] = np.nan
    x[0, 3] = np.nan
    x[0, 4, V - 1] = -3.0
    x[0, 5, V // 3] = -3.0e38
    token, parent = np.zeros((1, 6), dtype=np.int32), np.array([[-1, 0, 1, 2, 3, 4]], dtype=np.int32)
    logits = di.f32_to_bf16_bits(x) if dtype == "bf16" else x
    want = oracle.accept_path(logits, dtype, token, parent, 5)
    assert want[0].tolist() == [[0, 0, 0, 0, V - 1, V // 3]]
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    i32 = dict(dtype=torch.int32, device="cuda")
    for off in (0, 1):
        buf = torch.empty(x.size + off, dtype=tdt, device="cuda")
        lg = buf[off:].view(x.shape).copy_(torch.from_numpy(x))
        got = [torch.full((1, 6), -7, **i32), torch.full((1,), -7, **i32), torch.full((1, 6), -7, **i32), torch.full((1,), -7, **i32)]
        dream.dream_accept_path(lg, dream.BF16 if dtype == "bf16" else dream.F32, 1, 6, V, torch.from_numpy(token).cuda(), torch.from_numpy(parent).cuda(), 5, *got,
                                dream.alloc_workspace(dream.dream_accept_path_workspace(1, 6, V)))
        for g, w, what in zip(got, want, ("node_argmax", "accept_len", "accept_path", "bonus_token")):
            assert np.array_equal(g.cpu().numpy(), w), (what, off)


def test_duplicate_siblings_chain_and_single_node(gu):
    parent = np.array([[-1, 0, 0, 1, 2]], dtype=np.int32)
    token = np.array([[0, 5, 5, 6, 6]], dtype=np.int32)
    logits = np.zeros((1, 5, 8), dtype=np.float32)
    logits[0, 0, 5] = 1
    logits[0, 1, 6] = 1
    logits[0, 2, 6] = 1
    logits[0, 3, 2] = 1
    got = _compare(gu, logits, "f32", token, parent, 4)
    assert got[2][0].tolist() == [0, 1, 3, -1, -1]
    # chain deeper than max_depth
    parent = di.chain_tree(9)[None]
    token = np.ones((1, 9), dtype=np.int32)
    logits = np.zeros((1, 9, 4), dtype=np.float32)
    logits[0, :, 1] = 1
    got = _compare(gu, logits, "f32", token, parent, 6)
    assert got[1][0] == 6
    got = _compare(gu, logits[:, :1], "f32", token[:, :1], parent[:, :1], 6)
    assert got[1][0] == 0


def test_large_tree_of_1024_nodes(gu):
    T = 1024
    parent = di.random_tree(T, 12, 77)
    token = di.tree_tokens(parent, 50, 78)
    logits = di.normal((1, T, 50), "bf16", 79, di.STREAM_LOGITS)
    _compare(gu, logits, "bf16", token[None], parent[None], 12)


def test_parent_array_with_cycles_still_terminates(gu):
    """Device metadata is trusted, but a malformed parent array must end in unspecified results, not in a hang."""
    T, V = 8, 16
    parent = np.array([[-1, 1, 3, 2, 9, 4, -5, 0]], dtype=np.int32)      # self loop, 2<->3 cycle, out of range, negative
    token = np.full((1, T), 3, dtype=np.int32)
    logits = np.zeros((1, T, V), dtype=np.float32)
    logits[0, :, 3] = 1                                                     # every edge "matches"
    am, alen, path, bonus = gu.run_accept(logits, "f32", token, parent, 6)
    assert (am == 3).all() and 0 <= alen[0] <= 6 and bonus[0] == 3
    assert ((path >= -1) & (path < T)).all()
    assert alen[0] == 1 and path[0].tolist()[:2] == [0, 7]                  # only node 7 has a well-formed path


@pytest.mark.parametrize("chunks", [1, 2, 3, 5, 9, 17, 33, 65, 130])
def test_chunks_merged_by_every_number_of_lanes(gu, chunks):
    """1 to 64 lanes merge the chunks of a node (one of them has two or three of more than 64): the maximum in any chunk, and the same in a later one."""
    T, vocab = max(3, min(chunks, 40)), 8192 * (chunks - 1) + 5
    parent = di.random_tree(T, 4, 7)
    logits = di.normal((1, T, vocab), "f32", 71 + chunks, di.STREAM_LOGITS)
    token = np.zeros((1, T), dtype=np.int32)
    for i in range(T):
        at = (i * 7 + 3) % chunks
        for ch in (at, chunks - 1):
            logits[0, i, ch * 8192 + (i % 5)] = np.float32(9.0)
        if i:
            token[0, i] = (((parent[i] * 7 + 3) % chunks) * 8192 + parent[i] % 5 + (i % 3 == 2)) % vocab
    _compare(gu, logits, "f32", token, parent[None], 4)
