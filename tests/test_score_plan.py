"""How the two score passes of dream_visual_compress and dream_attention_entropy are cut into workgroups (csrc/score_plan.h, built for the host): every step of
every block is taken once, the splits are those that the stated cost picks, and the sizes of the GPU tests take the kernels that those tests are about."""
import ctypes
import math
import os
import random
import subprocess
import time

import pytest
from numpy import float32 as f32

from tests.test_gpu_compress import TWO_BLOCKS

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module", autouse=True)
def lib(tmp_path_factory):
    """tests/c/score_plan_check.cpp, which makes the header's plans."""
    out = str(tmp_path_factory.mktemp("plan") / "score_plan_check.so")
    root = os.path.dirname(HERE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-Werror", "-Wno-unknown-pragmas", "-I" + os.path.join(root, "paper_2505_19201_amd", "csrc"),
                    "-I" + os.path.join(root, "include"), os.path.join(HERE, "c", "score_plan_check.cpp"), "-o", out], check=True)
    global LIB
    LIB = ctypes.CDLL(out)
    LIB.score_workspace.restype = LIB.score_needs.restype = ctypes.c_longlong


FIELDS = ("ns1", "ns2", "units1", "units2", "wide1", "wide2", "order1", "order2", "blocks1", "blocks2")


def plan(B, H, D, n_q, n_keys, vis_start=0, v=0, with_pos=False, entropy=False, lse_given=False, direct=True):
    out = (ctypes.c_int * len(FIELDS))()
    LIB.score_plan(B, H, D, n_q, n_keys, vis_start, v, with_pos, entropy, lse_given, direct, out)
    return dict(zip(FIELDS, out))


def units(which, n):
    out = (ctypes.c_int * 3)()
    got = []
    for u in range(n):
        LIB.score_unit(which, u, out)
        got.append(tuple(out))
    return got


def ceil(a, b):
    return -(-a // b)


def lengths(which, n_q, n_keys, vis_start, v, with_pos):
    """Steps of 64 keys (pass 1) or rows (pass 2) that the blocks of 64 rows or keys see, longest first."""
    if which == 1:
        return sorted((ceil(n_keys if with_pos else min(64 * (i + 1), n_q, n_keys), 64) for i in range(ceil(n_q, 64))), reverse=True)
    rows = ceil(n_q, 64)
    return sorted((rows if with_pos else max(rows - (vis_start + 64 * i) // 64, 0) for i in range(ceil(max(v, 1), 64))), reverse=True)


def splits_by_cost(steps, heads, D, whole):
    """The longest run of steps of a workgroup, by the stated cost."""
    longest = max(steps[0], 1)
    if len(steps) * heads >= (512 if D == 256 else 768):
        return longest
    best, S = math.inf, longest
    for s in range(max(2, ceil(longest, 8)), max(longest, 2) + 1):
        wgs = sum(ceil(x, s) for x in steps) * heads
        cost = f32(3.0) * f32(ceil(wgs, 256)) + f32(1.2) * f32(s) - f32(whole if s == longest else 0.0)      # (as the plan rounds them: many are equal but for that)
        if wgs <= (512 if D == 256 else 1024) and cost < best:
            best, S = cost, s
    return S


def sample(seed):
    r = random.Random(seed)
    for _ in range(150):
        D, heads = r.choice((64, 128, 256)), r.choice((1, 2, 4, 7, 8, 16, 32, 64))
        B = r.choice((1, 1, 1, 2, 3, 8, 32))
        n_q = int(round(math.exp(r.uniform(0, math.log(9000)))))
        n_keys = n_q + r.choice((0, 0, 1, 64, 500))
        v = r.randint(1, min(n_keys, 3000))
        yield B, heads, D, n_q, n_keys, r.randint(0, n_keys - v), v, r.random() < 0.3, r.random() < 0.5


@pytest.mark.parametrize("seed", range(4))
def test_every_step_once_and_the_splits_of_least_cost(seed):
    for B, H, D, n_q, n_keys, vis_start, v, with_pos, entropy in sample(seed):
        p = plan(B, H, D, n_q, n_keys, vis_start, v, with_pos, entropy)
        for which in (1, 2):
            steps = lengths(which, n_q, n_keys, vis_start, v, with_pos)
            n, wide = p["units%d" % which], p["wide%d" % which]
            got = units(which, n)
            if wide:
                assert got == [(i, 0, 1) for i in range(ceil(len(steps), 2))]
                continue
            S = splits_by_cost(steps, H * B, D, 10.0 if entropy and which == 1 else 0.0)
            want = [(i, j, max(ceil(x, S), 1)) for i, x in enumerate(steps) for j in range(max(ceil(x, S), 1))]
            assert sorted(got) == want, (B, H, D, n_q, n_keys, vis_start, v, with_pos, which)
            assert max(k for _, _, k in got) <= p["ns%d" % which] <= 8
            if p["order%d" % which]:
                assert p["order%d" % which] == n
        assert LIB.score_needs() <= LIB.score_workspace(B, H, D, n_q, v)


def test_a_plan_is_made_in_no_time():
    """Every call makes one.  One head of 32768 rows and another of two million take microseconds (sums over all blocks for every number of steps: 500 us and minutes);
    a tenth of a millisecond leaves room for a busy machine."""
    for n in (32768, 1 << 21):
        best = math.inf
        for _ in range(10):
            start = time.perf_counter()
            plan(1, 1, 128, n, n, 0, 3000, entropy=True)
            best = min(best, time.perf_counter() - start)
        assert best < 1e-4


@pytest.mark.parametrize("B,H,D,n_q,ordered", [(1, 32, 128, 1279, True), (1, 16, 64, 6627, True), (8, 32, 64, 269, True), (16, 2, 128, 3084, True), (1, 16, 256, 1389, True), (1, 32, 256, 1619, False),
                                               (1, 16, 256, 4013, False), (1, 16, 256, 7417, False), (3, 4, 256, 5290, True), (8, 64, 256, 246, False), (1, 64, 128, 2100, False)])
def test_launches_with_an_order(B, H, D, n_q, ordered):
    """One sequence at head_dim 256 has an order of its workgroups only where all of them are at work together."""
    p = plan(B, H, D, n_q, n_q, entropy=True)
    assert (p["order1"] > 0) == ordered
    if ordered:
        assert 256 < p["units1"] * H * B <= (2048 if D != 256 else 512 if B == 1 else 1024)


@pytest.mark.parametrize("B,H,n_q,v,two", [(27, 16, 1280, 256, 1), (20, 16, 382, 327, 1), (12, 32, 376, 325, 1), (15, 8, 1033, 909, 0), (20, 4, 1211, 1140, 0), (13, 16, 1083, 305, 0), (9, 8, 1638, 1605, 0)])
def test_two_blocks_of_keys_at_head_dim_256(B, H, n_q, v, two):
    """Only where a CU's share of the steps is a good two times the longest block."""
    steps = lengths(2, n_q, n_q, 0, v, False)
    assert (10 * B * H * sum(steps) >= 21 * 512 * steps[0]) == two
    assert plan(B, H, 256, n_q, n_q, 0, v, lse_given=True)["wide2"] == two


@pytest.mark.parametrize("case", TWO_BLOCKS)
def test_sizes_of_the_gpu_test_take_workgroups_of_two_blocks(case):
    (B, Hq, _, D, P, v, vis_start), (sums, sums_own, entropies) = case
    for with_pos in (False, True):
        assert plan(B, Hq, D, P, P, vis_start, v, with_pos, lse_given=True)["wide2"] == sums
        own = plan(B, Hq, D, P, P, vis_start, v, with_pos)
        assert own["wide2"] == sums_own and own["wide1"] == entropies
        assert plan(B, Hq, D, P, P, with_pos=with_pos, entropy=True)["wide1"] == entropies
        other = plan(B, Hq, D, P, P, vis_start, v, with_pos, direct=False)       # what it is compared with
        assert not other["wide1"] and not other["wide2"]


def test_sizes_of_the_gpu_test_have_odd_and_even_numbers_of_blocks():
    sums, entropies = set(), set()
    for (B, Hq, _, D, P, v, _), (given, own, ent) in TWO_BLOCKS:
        sums |= {(D, ceil(v, 64) % 2)} if given and own else set()
        entropies |= {(D, ceil(P, 64) % 2)} if ent else set()
    assert sums == {(D, odd) for D in (64, 128, 256) for odd in (0, 1)}
    assert entropies == {(D, odd) for D in (128, 256) for odd in (0, 1)}
