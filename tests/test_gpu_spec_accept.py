"""GPU parity: dream_spec_accept (acceptance at a sampling temperature) against the float64 oracle.

The integers depend on float comparisons (u against a probability ratio, u against a cumulative sum).  The GPU
works in float32, so a sequence is compared only when the oracle's own run shows every such comparison clear of
float32 error -- decided on the CPU before the GPU result is looked at: |u - min(1, ratio)| > 1e-3 for every
acceptance test and the draw at least 2e-5 of the mass away from both ends of the drawn token's cumulative interval
(the float32 cumulative sums are good to about 1e-6 of the mass).
At least half of the sequences of every case must qualify, and all that qualify must match bit for bit.
A sequence that does not qualify is not waved through: its result must be one of the outcomes the oracle produces when
every too-close comparison on the way is resolved either way (the undecided acceptance tests flipped, the draw landing
on any token of positive probability whose cumulative interval is that close to the drawn point), enumerated on the CPU."""
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


RATIO_EPS, DRAW_EPS = 1e-3, 2e-5


def _clear(detail):
    ok = all(abs(u - min(1.0, r)) > RATIO_EPS for _, r, u in detail["tests"])
    return ok and detail["draw_margin"] > DRAW_EPS


def _legitimate_outcomes(tl64, dl64, token, parent, ua, ub, depth, inv_temperature, limit=64):
    """Every (accept_len, path, bonus) one sequence may legitimately yield: the oracle is re-run with each acceptance
    test that is within RATIO_EPS of its threshold taken either way (a flip changes the walk, so new close calls
    may appear: depth-first over them); the bonus may be any token of positive probability whose cumulative interval
    comes within DRAW_EPS of the drawn point."""
    outcomes, stack, seen = set(), [frozenset()], set()
    while stack and len(seen) < limit:
        flips = stack.pop()
        if flips in seen:
            continue
        seen.add(flips)
        alen, path, bonus, detail = oracle.spec_accept(tl64, dl64, token, parent, ua, ub, depth, inv_temperature=inv_temperature,
                                                       flip_nodes=flips, draw_window=DRAW_EPS)
        for node, ratio, u in detail[0]["tests"]:
            if abs(u - min(1.0, ratio)) <= RATIO_EPS and node not in flips:
                stack.append(flips | {node})
        for t in set(detail[0]["draw_window_tokens"]) | {int(bonus[0])}:
            outcomes.add((int(alen[0]), tuple(path[0].tolist()), t))
    return outcomes


def _draft_children(parent, dl_f64, g):
    """Children tokens drawn without replacement from the draft distribution of their parent (how a sampled draft
    tree is grown); the root's token is arbitrary."""
    B, T, V = dl_f64.shape
    token = np.zeros((B, T), dtype=np.int32)
    for b in range(B):
        for u in range(T):
            kids = np.flatnonzero(parent[b] == u)
            if kids.size:
                x = dl_f64[b, u]
                q = np.exp(x - x.max())
                q /= q.sum()
                token[b, kids] = g.choice(V, size=min(kids.size, V), replace=False, p=q)[:kids.size] if kids.size <= V else 0
    return token


def _formed_by_the_walk(B, T, V, dtype):
    """Whether the statistics of the nodes' rows are formed by the walk (the line of spec_accept.hip) and not beforehand."""
    nbytes = 2 * B * T * V * (4 if dtype == "f32" else 2)
    return nbytes * T >= 1200000000 if _small(B, T, V) else nbytes >= 60000000 and nbytes * T >= 3000000000


def _small(B, T, V):
    """Whether spec_walk_small_kernel takes the call: a workgroup per segment, of one chunk of 4096 or 8192 tokens, trees of up to 64 nodes."""
    return T <= 64 and any(-(-V // n) <= min(64, max(1, 256 // B)) for n in (4096, 8192))


def _branches(parent, detail, clear):
    """What happened at the nodes the compared sequences came to: accepted as which child, or all of how many rejected."""
    seen = set()
    for b in np.flatnonzero(clear):
        by_node = {}
        for node, ratio, u in detail[b]["tests"]:
            by_node.setdefault(int(parent[b, node]), []).append(u < min(1.0, ratio))
        for outcomes in by_node.values():
            if outcomes[-1]:
                seen.add(("accepted as child number", min(len(outcomes), 3)))
            else:
                seen.add(("all rejected, children", min(len(outcomes), 3)))
        if not by_node or all(o[-1] for o in by_node.values()):
            seen.add(("draw at a node without children",))
    return seen


def _case(gu, B, T, depth, V, dtype, seed, spread=2.0, noise=0.7, temperature=1.0, min_clear=0.5, min_compared=0, limit=None, never=0.0):
    """limit: depth limit of the call, below the tree's depth.  never: share of the nodes whose random number lets no test pass."""
    g = di.rng(seed, 700)
    parent = np.stack([di.random_tree(T, depth, seed, b) for b in range(B)]) if T > 1 else np.full((B, 1), -1, dtype=np.int32)
    t32 = di.normal((B, T, V), "f32", seed, di.STREAM_LOGITS) * np.float32(spread)
    d32 = t32 + di.normal((B, T, V), "f32", seed, di.STREAM_DRAFT_LOGITS) * np.float32(noise)
    tl = t32 if dtype == "f32" else di.f32_to_bf16_bits(t32)
    dl = d32 if dtype == "f32" else di.f32_to_bf16_bits(d32)
    tl64, dl64 = di.as_f64(tl, dtype), di.as_f64(dl, dtype)
    token = _draft_children(parent, dl64 / temperature, g)
    ua = g.uniform(size=(B, T)).astype(np.float32)
    ub = g.uniform(size=B).astype(np.float32)
    if never:
        ua[g.random(size=(B, T)) < never] = 2.0
    depth = depth if limit is None else limit
    want_len, want_path, want_bonus, detail = oracle.spec_accept(tl64, dl64, token, parent, ua.astype(np.float64), ub.astype(np.float64),
                                                                depth, inv_temperature=1.0 / temperature)
    clear = np.array([_clear(d) for d in detail])
    assert clear.mean() >= min_clear and clear.sum() >= min_compared, (clear.mean(), clear.sum())
    alen, path, bonus = gu.run_spec_accept(tl, dl, dtype, token, parent, ua, ub, depth, temperature)
    assert (alen >= 0).all() and (alen <= depth).all() and (bonus >= 0).all() and (bonus < V).all()
    assert np.array_equal(alen[clear], want_len[clear]), (alen[clear], want_len[clear])
    assert np.array_equal(path[clear], want_path[clear])
    assert np.array_equal(bonus[clear], want_bonus[clear])
    for b in np.flatnonzero(~clear):      # too close to call in float32: any resolution of the close calls is right, nothing else
        legit = _legitimate_outcomes(tl64[b:b + 1], dl64[b:b + 1], token[b:b + 1], parent[b:b + 1], ua[b:b + 1].astype(np.float64),
                                     ub[b:b + 1].astype(np.float64), depth, 1.0 / temperature)
        assert (int(alen[b]), tuple(path[b].tolist()), int(bonus[b])) in legit, (b, alen[b], path[b], bonus[b], legit)
    _case.last = (parent, detail, clear)
    return alen, clear


def test_worked_example(gu):
    p, q = np.array([0.5, 0.3, 0.2]), np.array([0.2, 0.5, 0.3])
    tl = np.log(p)[None, None].repeat(3, axis=1).astype(np.float32)
    dl = np.log(q)[None, None].repeat(3, axis=1).astype(np.float32)
    parent = np.array([[-1, 0, 0]], dtype=np.int32)
    for tok, ua, ub, want in (([9, 1, 0], [0, 0.5, 0.9], 0.3, (1, [0, 1])), ([9, 1, 0], [0, 0.7, 0.999], 0.3, (1, [0, 2])),
                              ([9, 1, 2], [0, 0.7, 0.0], 0.99, (0, [0, -1]))):
        alen, path, bonus = gu.run_spec_accept(tl, dl, "f32", np.array([tok]), parent, np.array([ua]), np.array([ub]), 6)
        assert alen[0] == want[0] and path[0, :2].tolist() == want[1] and path[0, 2:].tolist() == [-1] * 5
        if want[0] == 0:
            assert bonus[0] == 0
    for u, want in ((0.0, 0), (0.49, 0), (0.51, 1), (0.79, 1), (0.81, 2), (0.999, 2)):
        _, _, bonus = gu.run_spec_accept(tl[:, :1], dl[:, :1], "f32", np.array([[9]]), np.array([[-1]], dtype=np.int32),
                                         np.array([[0.0]]), np.array([u]), 6)
        assert bonus[0] == want


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_cold_limit_is_the_greedy_rule(gu, dtype):
    cfg = di.Config("s", dtype, 8, 4, 4, 64, 256, 8, 8, 40, 5, 1, 2, 5000, 1, 71)
    logits, token, parent, _ = di.accept_inputs(cfg)
    dlog = di.normal(logits.shape, dtype, 72, di.STREAM_DRAFT_LOGITS)
    want_am, want_len, want_path, want_bonus = oracle.accept_path(logits, dtype, token, parent, cfg.depth)
    g = di.rng(73, 701)
    alen, path, bonus = gu.run_spec_accept(logits, dlog, dtype, token, parent, g.uniform(size=token.shape), g.uniform(size=cfg.batch),
                                           cfg.depth, temperature=1.0 / 400.0)
    # a row whose maximum is shared by two tokens (bf16 is coarse) is a fair coin for the sampling rule but not for
    # the greedy one: compare the sequences whose visited rows have a unique maximum
    f = di.as_f64(logits, dtype)
    unique = np.array([all((f[b, n] == f[b, n].max()).sum() == 1 for n in want_path[b] if n >= 0) for b in range(cfg.batch)])
    assert unique.sum() >= cfg.batch // 2
    assert np.array_equal(alen[unique], want_len[unique]) and np.array_equal(path[unique], want_path[unique])
    assert np.array_equal(bonus[unique], want_bonus[unique])


@pytest.mark.parametrize("V", [1, 5, 1000, 1024, 1025, 32003])
def test_ragged_vocabularies(gu, V):
    _case(gu, 16, min(13, max(2, V)), 4, V, "f32", 800 + V)


@pytest.mark.parametrize("dtype,temperature", [("f32", 1.0), ("bf16", 1.0), ("bf16", 0.7)])
def test_trees_of_the_paper_shape(gu, dtype, temperature):
    alen, clear = _case(gu, 48, 33, 6, 4000, dtype, 900, temperature=temperature)
    assert len(set(alen[clear].tolist())) >= 3          # several different accepted depths occur


@pytest.mark.parametrize("name", ["llava", "gemma3"])
def test_full_size_vocabularies(gu, name):
    cfg = di.CONFIGS[name]
    # (at 262144 tokens an interval of the cumulative sum is a few 1e-6 of the mass wide, so few draws are DRAW_EPS clear
    # of both ends: the batch is sized so that at least 8 sequences are compared bit for bit all the same)
    _case(gu, 12 if cfg.vocab <= 65536 else 36, cfg.n_tree, cfg.depth, cfg.vocab, "bf16", cfg.seed, min_clear=0.2, min_compared=8)


def test_largest_tree(gu):
    """1024 nodes per sequence, the most the entry point takes (every per-node table at its full size)."""
    _case(gu, 3, 1024, 12, 777, "f32", 960)


def test_every_branch_of_the_walk_is_exercised(gu):
    """The kernel treats the first rejection at a node symbolically, the second by building arrays, and draws in
    three different ways; the oracle's record of the tests says which of these each compared sequence took."""
    _case(gu, 96, 33, 6, 4000, "bf16", 950, noise=1.0)
    parent, detail, clear = _case.last
    seen = _branches(parent, detail, clear)
    want = {("accepted as child number", 1), ("accepted as child number", 2), ("accepted as child number", 3),
            ("all rejected, children", 1), ("all rejected, children", 2), ("all rejected, children", 3),
            ("draw at a node without children",)}
    assert want <= seen, want - seen


@pytest.mark.parametrize("V", [8192, 8193, 24577, 65536, 540001])
@pytest.mark.parametrize("polls", [0, -1])
def test_workgroups_of_a_sequence(gu, V, polls):
    """Rows of 2, 3, 7, 16 and (of 16384) 33 chunks of 4096 tokens, summed by several workgroups that exchange their
    sums, and (polls < 0: nobody waits) by workgroup 0 in the others' place."""
    import paper_2505_19201_amd as dream
    dream.dream_set_accept_spin(polls)
    try:
        _case(gu, 3 if V > 100000 else 8, 21, 5, V, "f32", 970 + V, noise=1.0, min_clear=0.0)
    finally:
        dream.dream_set_accept_spin(0)


@pytest.mark.parametrize("B,T,V", [(40, 6, 40000), (64, 4, 60000), (100, 3, 20000), (20, 5, 262145), (300, 3, 9001)])
@pytest.mark.parametrize("polls", [0, -1])
def test_shares_of_a_workgroup(gu, B, T, V, polls):
    """Two and four times as many logits in a workgroup's registers, more than they hold, one workgroup per sequence; with the statistics of all
    nodes formed beforehand (test_statistics_formed_by_the_walk has them formed by the walk)."""
    assert not _formed_by_the_walk(B, T, V, "f32")
    import paper_2505_19201_amd as dream
    dream.dream_set_accept_spin(polls)
    try:
        _case(gu, B, T, 3, V, "f32", 1970 + V, noise=1.0, min_clear=0.0)
    finally:
        dream.dream_set_accept_spin(0)


@pytest.mark.parametrize("polls", [0, -1])
@pytest.mark.parametrize("B,T,V,dtype,temperature", [
    (4, 60, 40000, "f32", 1.0), (8, 60, 40003, "bf16", 0.7),                # a chunk of 4096 logits a workgroup
    (16, 33, 70000, "f32", 0.7), (32, 24, 80000, "bf16", 1.0),              # of 8192, of 16384
    (64, 16, 70000, "bf16", 1.0), (260, 16, 17001, "bf16", 1.0),             # more segments than workgroups; one workgroup, no exchange
    (2, 21, 1060001, "f32", 1.0)])                                          # two chunks a segment
def test_statistics_formed_by_the_walk(gu, B, T, V, dtype, temperature, polls):
    """Many logits: the walk works out the statistics of a node's rows when it comes to the node.  Every share of a workgroup, both types, with the
    exchange and without; then a depth limit inside the tree, so that walks end at nodes with children and draw from the masses of that
    round."""
    import paper_2505_19201_amd as dream
    assert _formed_by_the_walk(B, T, V, dtype)
    dream.dream_set_accept_spin(polls)
    try:
        if polls == 0:
            _case(gu, B, T, 5, V, dtype, 2970 + V, noise=1.0, temperature=temperature, min_clear=0.0)
        alen, clear = _case(gu, B, T, 5, V, dtype, 2971 + V, noise=0.5, temperature=temperature, min_clear=0.0, limit=2)
        assert alen.max() == 2
    finally:
        dream.dream_set_accept_spin(0)


@pytest.mark.parametrize("polls", [0, -1])
@pytest.mark.parametrize("B,T,V,dtype", [(1, 5, 1048577, "f32"), (2, 6, 1060003, "bf16")])
def test_segments_of_two_chunks_with_statistics_beforehand(gu, B, T, V, dtype, polls):
    """More than 64 chunks of 16384 tokens: a segment is two of them, the last one alone in its segment or not."""
    import paper_2505_19201_amd as dream
    assert not _formed_by_the_walk(B, T, V, dtype)
    dream.dream_set_accept_spin(polls)
    try:
        for i in range(3):
            _case(gu, B, T, 3, V, dtype, 4970 + V + i, noise=1.0, min_clear=0.0)
    finally:
        dream.dream_set_accept_spin(0)


@pytest.mark.parametrize("polls", [0, -1])
def test_every_branch_with_statistics_formed_by_the_walk(gu, polls):
    """Accepted as first, second and third child, all of one, two and three children rejected, a walk that ends at a leaf."""
    import paper_2505_19201_amd as dream
    B, T, V = 96, 33, 9000
    assert _formed_by_the_walk(B, T, V, "f32")
    dream.dream_set_accept_spin(polls)
    try:
        _case(gu, B, T, 6, V, "f32", 953, noise=1.0)
    finally:
        dream.dream_set_accept_spin(0)
    assert _branches(*_case.last) >= {(what, n) for what in ("accepted as child number", "all rejected, children") for n in (1, 2, 3)} | \
        {("draw at a node without children",)}


@pytest.mark.parametrize("polls", [0, -1])
@pytest.mark.parametrize("B,T,V,dtype", [(6, 33, 4000, "f32"), (8, 60, 20000, "f32"), (16, 33, 70000, "bf16")])
def test_a_draft_equal_to_the_target(gu, B, T, V, dtype, polls):
    """Equal rows leave no residual behind a rejection (which the random numbers force): the target stays as it is and the rejected token leaves the
    draft.  The smallest with the statistics formed beforehand, the others with those of the walk."""
    import paper_2505_19201_amd as dream
    assert _formed_by_the_walk(B, T, V, dtype) == (V > 4000)
    dream.dream_set_accept_spin(polls)
    try:
        _case(gu, B, T, 5, V, dtype, 3970 + V, noise=0.0, never=0.5, min_clear=0.25)
    finally:
        dream.dream_set_accept_spin(0)
    parent, detail, clear = _case.last
    assert any(u > 1.0 for b in np.flatnonzero(clear) for _, _, u in detail[b]["tests"])


@pytest.mark.parametrize("V", [1000, 24577, 65536])
@pytest.mark.parametrize("offset", [1, 4, 72, 255])
def test_workspace_at_any_address(gu, V, offset):
    """The workgroups of a sequence exchange 64-bit words in the workspace, which may start at any byte: same results as with an aligned
    one, and nothing written outside the bytes handed over."""
    import torch
    import paper_2505_19201_amd as dream
    B, T, depth = 4, 21, 5
    g = di.rng(980 + V, 700)
    parent = np.stack([di.random_tree(T, depth, 981, b) for b in range(B)])
    t32 = di.normal((B, T, V), "f32", 982, di.STREAM_LOGITS) * np.float32(2.0)
    d32 = t32 + di.normal((B, T, V), "f32", 983, di.STREAM_DRAFT_LOGITS)
    token = _draft_children(parent, d32.astype(np.float64), g)
    ua, ub = g.uniform(size=(B, T)).astype(np.float32), g.uniform(size=B).astype(np.float32)
    want = gu.run_spec_accept(t32, d32, "f32", token, parent, ua, ub, depth)
    need = dream.dream_spec_accept_workspace(B, T, V)
    buf = torch.full((offset + need + 300,), 0xFF, dtype=torch.uint8, device="cuda")
    dev = [dream.to_device(np.ascontiguousarray(a)) for a in (t32, d32, token.astype(np.int32), parent.astype(np.int32), ua, ub)]
    out = [torch.full(s, -7, dtype=torch.int32, device="cuda") for s in ((B,), (B, depth + 1), (B,))]
    dream.dream_spec_accept(dev[0], dev[1], dream.F32, B, T, V, dev[2], dev[3], dev[4], dev[5], depth, 1.0, *out, buf[offset:offset + need])
    torch.cuda.synchronize()
    for got, w in zip(out, want):
        assert np.array_equal(got.cpu().numpy(), w)
    outside = torch.cat([buf[:offset], buf[offset + need:]])
    assert (outside == 0xFF).all()


@pytest.mark.parametrize("V,dtype", [(24577, "f32"), (65536, "bf16"), (131072, "f32")])
def test_whoever_sums_a_segment_the_result_is_the_same(gu, V, dtype):
    """Every result, close calls included, is the same whether the workgroups exchange their sums or workgroup 0 forms them all
    (polls < 0): one sum kept in registers from rejection to rejection, the other recomputed from the logits.  Identical draft and
    target rows but for a few tokens make the masses small and the comparisons close."""
    import paper_2505_19201_amd as dream
    B, T, depth = 16, 33, 6
    g = di.rng(990 + V, 700)
    parent = np.stack([di.random_tree(T, depth, 991, b) for b in range(B)])
    t32 = di.normal((B, T, V), "f32", 992, di.STREAM_LOGITS) * np.float32(2.0)
    d32 = t32 + di.normal((B, T, V), "f32", 993, di.STREAM_DRAFT_LOGITS) * (g.random((B, T, 1)) < 0.7).astype(np.float32)
    tl, dl = (t32, d32) if dtype == "f32" else (di.f32_to_bf16_bits(t32), di.f32_to_bf16_bits(d32))
    token = np.argsort(-t32[:, 0], axis=1)[:, :T].astype(np.int32)            # likely tokens, so that siblings are rejected one after the other
    ua, ub = g.uniform(0.5, 1.0, size=(B, T)).astype(np.float32), g.uniform(size=B).astype(np.float32)
    want = gu.run_spec_accept(tl, dl, dtype, token, parent, ua, ub, depth)
    dream.dream_set_accept_spin(-1)
    try:
        got = gu.run_spec_accept(tl, dl, dtype, token, parent, ua, ub, depth)
    finally:
        dream.dream_set_accept_spin(0)
    for a, b in zip(got, want):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("B,T,V,dtype,small", [
    (3, 64, 4096, "f32", True), (3, 65, 4097, "f32", False),    # the largest tree of spec_walk_small_kernel and the next; one segment of one chunk, two with one token in the last
    (2, 1, 9000, "bf16", True), (2, 2, 8200, "f32", True),      # no test at all; one
    (4, 64, 40000, "f32", True), (4, 65, 40000, "f32", False), (4, 64, 40003, "bf16", True), (20, 30, 70000, "bf16", True),   # statistics formed by the walk; rows off the 16-byte boundaries; 8192 tokens a workgroup
    (64, 40, 16384, "f32", True), (65, 40, 16384, "f32", True),        # 256 workgroups of 4096 tokens; 130 of 8192
    (80, 12, 25000, "bf16", False), (130, 9, 8200, "f32", False)])     # more chunks of 8192 tokens than workgroups of a sequence: two workgroups, and one
@pytest.mark.parametrize("limit", [5, 2, 0])
def test_both_walks_give_the_same(gu, B, T, V, dtype, small, limit):
    """Trees, rows and batches on both sides of the lines between the two walks, close calls included: the same whether the workgroups exchange their sums or (polls < 0) workgroup 0
    forms them all, which is spec_walk_kernel's way; down to a depth limit of 0, where a root with children is drawn from."""
    assert _small(B, T, V) == small
    import paper_2505_19201_amd as dream
    g = di.rng(5990 + V + T, 700)
    parent = np.stack([di.random_tree(T, 5, 5991, b) for b in range(B)]) if T > 1 else np.full((B, 1), -1, dtype=np.int32)
    t32 = di.normal((B, T, V), "f32", 5992, di.STREAM_LOGITS) * np.float32(2.0)
    d32 = t32 + di.normal((B, T, V), "f32", 5993, di.STREAM_DRAFT_LOGITS)
    token = _draft_children(parent, d32.astype(np.float64), g)
    tl, dl = (t32, d32) if dtype == "f32" else (di.f32_to_bf16_bits(t32), di.f32_to_bf16_bits(d32))
    ua, ub = g.uniform(0.2, 1.0, size=(B, T)).astype(np.float32), g.uniform(size=B).astype(np.float32)
    got = gu.run_spec_accept(tl, dl, dtype, token, parent, ua, ub, limit)
    dream.dream_set_accept_spin(-1)
    try:
        want = gu.run_spec_accept(tl, dl, dtype, token, parent, ua, ub, limit)
    finally:
        dream.dream_set_accept_spin(0)
    for a, b in zip(got, want):
        assert np.array_equal(a, b)
    assert got[0].max() <= limit and (got[2] >= 0).all() and (got[2] < V).all()
