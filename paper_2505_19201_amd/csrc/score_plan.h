// How the two score passes of compress.hip are cut into workgroups: plain integer arithmetic, also compiled for the host by the test of these plans.
#pragma once
#include "dream.h"
#include "sizes.h"
#include <algorithm>
#include <cmath>

namespace dream {

constexpr int COLS = 32;           // held rows or keys of a wave (64 halve the loads per score and measured 5-20 % slower: fewer workgroups)
constexpr int BLOCK = 2 * COLS;    // of a workgroup: two column slots
constexpr int STEP = 64;           // rows per step
constexpr int MAX_SPLITS = 8;

// Which blocks are split how often.  The causal triangle gives the blocks of a pass different numbers of steps; a block with
// more than `S` of them is divided evenly over several workgroups, so that no workgroup of the launch walks more than S.
// rank: position of a block when they are sorted by falling length; the first count[j] of them have a split j.
struct SplitMap {
    int32_t count[MAX_SPLITS];
};
struct SplitUnit {
    int rank, split, n;     // block (by rank), its split, and how many splits it has
};
// The units of a launch of a few rounds of workgroups at most, in the order of dispatch: 16 bits each, block * 64 + split * 8 + splits - 1.  See order_units().
constexpr int MAX_ORDERED = 128, MAX_ORDERED_BLOCKS = 1024;
struct UnitOrder {
    int32_t n;              // units, or 0: the order of the map
    uint32_t pair[MAX_ORDERED / 2];
};
// Unit u of a launch: by its pair of the order if that is an `ordered` one, else by the map
__attribute__((always_inline)) constexpr SplitUnit split_unit(const SplitMap &map, bool ordered, uint32_t pair, int u)
{
    const uint32_t e = pair >> (u & 1) * 16;
    SplitUnit r = {u, 0, 0};
#pragma unroll
    for (int j = 0; j < MAX_SPLITS - 1; j++)
        if (r.split == j && r.rank >= map.count[j]) {
            r.rank -= map.count[j];
            r.split = j + 1;
        }
#pragma unroll
    for (int j = 0; j < MAX_SPLITS; j++)
        r.n += r.rank < map.count[j];
    return {ordered ? (int)(e >> 6 & (MAX_ORDERED_BLOCKS - 1)) : r.rank, ordered ? (int)(e >> 3 & 7) : r.split, ordered ? (int)(e & 7) + 1 : r.n};
}

// Blocks are split while the launch would have fewer workgroups than this: two or three per CU.
inline int resident_groups(int head_dim) { return head_dim == 256 ? 512 : 768; }

// Steps of 64 keys or rows that the blocks of a pass have, longest first: all the same, or (falls) one less from block to block down to none.
struct BlockSteps {
    int first;
    bool falls;
    int operator()(int rank) const { return falls ? std::max(first - rank, 0) : first; }
    // all steps of `blocks` blocks
    int64_t total(int blocks) const
    {
        const int64_t n = falls ? std::max(std::min(blocks, first), 0) : blocks;
        return n * first - (falls ? n * (n - 1) / 2 : 0);
    }
    // of `blocks` blocks, those with more than n steps
    int longer_than(int n, int blocks) const { return falls ? std::min(std::max(first - n, 0), blocks) : first > n ? blocks : 0; }
    // workgroups of at most S steps that `blocks` blocks make
    int64_t workgroups(int S, int blocks) const
    {
        if (!falls)
            return (int64_t)blocks * ceil_div(first, S);
        auto up_to = [S](int64_t n) {              // of blocks of 1, 2, .. n steps
            const int64_t whole = n > 0 ? n / S : 0, rest = n > 0 ? n % S : 0;
            return S * (whole * (whole + 1) / 2) + rest * (whole + 1);
        };
        return up_to(first) - up_to((int64_t)first - blocks);
    }
};

// Splits of one pass.  `heads`: workgroups per unit (heads times sequences); `resident`: see above.  If the blocks as they are already fill the chip, they stay whole.  Otherwise a block is divided over workgroups of at
// most S steps, two at least and at most 8 workgroups a block, with the S of least 3 R + 1.2 S, R = ceil(workgroups / 256): a workgroup that shares
// its CU costs it about three steps (its own first loads and its end), and the longest one runs its steps one after the other, a step at 1.2
// of what it takes of a CU's time when others fill the gaps.  At most four workgroups a CU are at work together (two at head_dim 256), and more were always slower.
// `whole`: what a launch with whole blocks is worth, in these units: without partial values the entropies need one launch less
// (all launches, us, split / whole: LLaVA 704 rows 13.7 / 13.4, 2 x 500 Pixtral rows 14.9 / 12.2; whole before / now: SmolVLM 1600 rows 22.1 / 20.6).
// Entropy of one prompt, us, by S (all its launches, units in the order below): Pixtral 1279 rows 9 21.4, 10 20.1, 13 19.8, 16 20.5, 20 21.6; LLaVA 704
// rows 3 14.8, 4 15.3, 5 14.7, 6 13.7, 7 14.0, 9 15.0; Gemma3 1280 rows 9 20.5, 10 19.2, 12 20.8, 16 23.8.  The rule takes 10, 6 and 10.
// Every call makes its plan, so nothing here goes over the blocks once per S: with that it took 500 us of the host for one head of 32768 rows, 1.3 us for 32 heads of 704 (both passes, order
// included), now 0.6 and 0.5, and the entropy of one head of 16384 rows took 84 us, now 49.
inline int plan_splits(int blocks, int64_t heads, int resident, float whole, BlockSteps len, SplitMap *map, int *units)
{
    const int longest = len(0) > 1 ? len(0) : 1;
    int S = longest;
    if ((int64_t)blocks * heads < resident) {
        float best = INFINITY;
        const int64_t together = resident > 512 ? 1024 : 512;
        auto take_if_best = [&](int s) {
            const int64_t wgs = len.workgroups(s, blocks) * heads;
            const float cost = 3.0f * ceil_div(wgs, 256) + 1.2f * s - (s == longest ? whole : 0.0f);
            if (wgs <= together && cost < best) {
                best = cost;
                S = s;
            }
        };
        for (int s = std::max(2, ceil_div(longest, MAX_SPLITS)); s < longest && 3.0f + 1.2f * s < best; s++)      // (a launch has one workgroup at least)
            take_if_best(s);
        take_if_best(std::max(longest, 2));
    }
    int most = 1;
    *units = 0;
    for (int j = 0; j < MAX_SPLITS; j++) {
        map->count[j] = j == 0 ? blocks : len.longer_than(j * S, blocks);
        *units += map->count[j];
        if (map->count[j] > 0)
            most = j + 1;
    }
    int pow2 = 1;   // 1, 2, 4 or 8: pass 2 is compiled for these counts of pass-1 splits
    while (pow2 < most)
        pow2 *= 2;
    return pow2;
}

// Order of dispatch of a launch of a few rounds of workgroups at most.  Workgroup i starts on CU i mod 256, `heads` workgroups to a unit, so units 256 / heads
// apart share a CU, all of them until the end of the launch where they are at work together: the longest go first, and every further round gives its longest to the CU with the fewest
// steps so far.
//
// Up to how many workgroups (order_limit()).  Without an order one sequence goes longest block first, and each workgroup to the CU that is first free; several sequences go one after the other, and
// the long blocks of the last one come when the CUs run empty.  At head_dim 64 and 128 four workgroups share a CU and an order pays up to 2048.  us, no order / order, by the number of workgroups:
// one sequence, entropy: 960 22.8 / 21.5, 1120 27.5 / 25.2, 1152 36.7 / 35.8, 1328 63.5 / 60 and 82 / 83, 1664 90.7 / 87, 1712 126 / 126; column sums: 1216 34.5 / 34.8, 1408 36.6 / 35.7, 1888 67.2 / 65.2;
// several, entropy: 640 10.4 / 9.1, 1024 21.0 / 14.3, 1200 58 / 49, 1568 75 / 60, 1792 31.9 / 27, 2048 19.5 / 17.5; column sums: 1024 23.6 / 20.3, 1408 52.8 / 38.5, 1536 23.5 / 19.5, 1920 65.6 / 67.2,
// 2048 48.6 / 38.9.  At head_dim 256 two share a CU.  One sequence: an order that is not over after 512 takes the choice from CUs that would have made it better: 364 60.9 / 58.7, 384 29.6 / 28.5,
// 512 30.1 / 29.6, 656 48.0 / 48.4, 752 102 / 102, 832 35 / 40, 896 (both passes) 49.4 / 54.0, 1024 82 / 90, 1856 241 / 260.  Several sequences: 640 28.7 / 24.4, 924 112 / 103, 996 129 / 120,
// 1024 25.0 / 24.2, 1152 48.6 / 43.5, 1200 51.8 / 47.5, 1280 27.1 / 28.1 and 52.3 / 42.5, 2016 66 / 67, 2048 29.6 / 31.7 and 118 / 96: up to 1024.
inline int order_limit(int head_dim, int batch) { return head_dim != 256 ? 2048 : batch == 1 ? 512 : 1024; }

inline void order_units(int64_t heads, int units, int limit, BlockSteps len, const SplitMap &map, UnitOrder *order)
{
    order->n = 0;
    if (units > MAX_ORDERED || units < 2 || map.count[0] > MAX_ORDERED_BLOCKS || units * heads > limit || units * heads <= 256)
        return;
    struct Unit { int steps; uint32_t code; } unit[MAX_ORDERED];
    int n = 0;
    for (int r = 0; r < map.count[0]; r++) {
        int of = 0;
        while (of < MAX_SPLITS && r < map.count[of])
            of++;
        const int all = len(r), each = ceil_div(all, of);
        for (int j = 0; j < of; j++)
            unit[n++] = {std::max(std::min(each, all - j * each), 0), (uint32_t)(r << 6 | j << 3 | (of - 1))};
    }
    std::sort(unit, unit + n, [](const Unit &x, const Unit &y) { return x.steps != y.steps ? x.steps > y.steps : x.code < y.code; });
    const int bins = std::min(std::max((int)(256 / heads), 1), n), rounds = ceil_div(n, bins);
    int load[MAX_ORDERED], by_load[MAX_ORDERED], dealt[2 * MAX_ORDERED];      // dealt: the unit that round t gives bin i, at t * bins + i
    for (int i = 0; i < bins; i++) {
        load[i] = 0;
        by_load[i] = i;
    }
    for (int t = 0; t < rounds; t++) {
        std::sort(by_load, by_load + bins, [&](int x, int y) { return load[x] != load[y] ? load[x] < load[y] : x < y; });
        for (int i = 0; i < std::min(bins, n - t * bins); i++) {
            load[by_load[i]] += unit[t * bins + i].steps;
            dealt[t * bins + by_load[i]] = t * bins + i;
        }
    }
    // the last round may be short: its bins come first in every round (by_load still says in which order it was dealt)
    for (int i = 0; i < MAX_ORDERED / 2; i++)
        order->pair[i] = 0;
    for (int u = 0; u < n; u++)
        order->pair[u >> 1] |= unit[dealt[u / bins * bins + by_load[u % bins]]].code << (u & 1) * 16;
    order->n = n;
}

// Workgroups of two blocks (SLOTS = 4) in the place of one, where the blocks are whole and in the order of the map.  A wave then takes whole steps: half the barriers,
// loads and first steps per score.  It pays where workgroups that are half as many still come to several rounds.  us, one block / two, by their number (of two), all launches:
// column sums, head_dim 64: 1440 57.6 / 58.5, 1728 63.7 / 63.3, 2016 72.1 / 73.3, 2304 79.0 / 78.8, 3072 45.0 / 43.2, 4608 128.4 / 125.6; 128: 1024 52.2 / 56.0,
// 1280 43.6 / 44.0 and 68.9 / 65.9, 1440 98.5 / 90.7, 1920 57.1 / 55.9, 4096 148.7 / 129.7; 256: 640 131.8 / 122.0, 1024 138.2 / 116.4, 2048 272 / 243 (fewer are dealt to the CUs).
// Sums at head_dim 256 from 600 on and only where a CU's share of the steps is at least 2.1 times the longest block: below that the end of the launch, when the last of these workgroups run alone, costs more than
// they save.  By that ratio: 1.55 61.7 / 66.8, 1.8 59.0 / 61.0, 1.9 80.9 / 81.8, 2.07 64.7 / 69.0, 2.1 30.2 / 29.6, 2.2 39.7 / 36.0, 2.4 67.0 / 65.5, 2.5 72.1 / 63.8, 2.6 42.9 / 40.0, 3.1 109 / 92, 3.0 201 / 205, 3.4 51.5 / 49.6.
// Log-sum-exps (entropy), 128: 1152 29.6 / 33.1 and 74.0 / 63.6, 1536 62.6 / 64.8, 1760 68.1 / 68.4, 1920 44.3 / 45.8, 2304 74.8 / 72.3, 3072 65.9 / 64.3 but with 5 steps 39.7 / 40.7,
// 5120 160 / 148; 256: 832 60.3 / 63.7, 1024 51.7 / 52.1, 1280 60.4 / 60.1 and 52.2 / 47.6, 1824 177 / 160, 2560 152 / 134; 64: 3328 91.6 / 93.4, 4096 39.8 / 44.6, 6656 169.8 / 165.4: one block.
inline bool take_double(bool want, const UnitOrder &order, SplitMap *map, int *units)
{
    if (!want || order.n || *units != map->count[0])
        return false;
    *units = map->count[0] = ceil_div(map->count[0], 2);
    return true;
}

struct CompressPlan {
    int n_q_pad, ns1, ns2;
    int units1, units2;            // (block, split) units of the two passes
    SplitMap map1, map2;
    UnitOrder order1, order2;
    bool wide1, wide2;             // workgroups of twice a block
    size_t off_lse, off_part;
};

// `with_pos`: rows come with explicit positions, so any block may have to walk everything
inline CompressPlan compress_plan(int batch, int n_heads, int head_dim, int n_q, int n_keys, int vis_start, int vis_len, int dtype, bool with_pos, bool entropy, bool lse_given, bool direct)
{
    CompressPlan p;
    p.n_q_pad = (n_q + 15) / 16 * 16;
    p.ns1 = p.ns2 = 1;
    p.units1 = p.units2 = 1;
    p.order1.n = p.order2.n = 0;
    p.wide1 = p.wide2 = false;
    if (dtype == DREAM_BF16) {
        const int resident = resident_groups(head_dim);
        const int b1 = ceil_div(n_q, BLOCK), b2 = ceil_div(vis_len > 0 ? vis_len : 1, BLOCK), rows = ceil_div(n_q, 64);
        const int64_t heads = (int64_t)n_heads * batch;
        // (without positions there are no more rows than keys)
        const BlockSteps len1 = {with_pos ? ceil_div(n_keys, STEP) : b1, !with_pos}, len2 = {with_pos ? rows : rows - vis_start / STEP, !with_pos};
        p.ns1 = plan_splits(b1, heads, resident, entropy ? 10.0f : 0.0f, len1, &p.map1, &p.units1);
        p.ns2 = plan_splits(b2, heads, resident, 0.0f, len2, &p.map2, &p.units2);
        order_units(heads, p.units1, order_limit(head_dim, batch), len1, p.map1, &p.order1);
        order_units(heads, p.units2, order_limit(head_dim, batch), len2, p.map2, &p.order2);
        if (direct) {
            const int64_t wgs1 = ceil_div(b1, 2) * heads, wgs2 = ceil_div(b2, 2) * heads;
            p.wide1 = take_double(head_dim == 256 ? wgs1 >= 1280 : head_dim == 128 && wgs1 >= 2300 && len1(0) >= 8, p.order1, &p.map1, &p.units1);
            const bool many2 = head_dim == 64 ? wgs2 >= 2048 : head_dim == 128 ? wgs2 >= 1400 : wgs2 >= 600 && 10 * heads * len2.total(b2) >= 21 * 512 * (int64_t)len2(0);
            p.wide2 = take_double((p.ns1 == 1 || lse_given) && many2, p.order2, &p.map2, &p.units2);
        }
    }
    p.off_lse = DREAM_WORKSPACE_MIN_BYTES;
    p.off_part = align_up(p.off_lse + (size_t)p.ns1 * batch * n_heads * p.n_q_pad * sizeof(float), 256);
    return p;
}

// The most splits a plan of these sizes takes, whatever the keys and positions are (the workspace query knows neither).
inline int most_splits(int64_t blocks, int64_t heads, int head_dim, int dtype)
{
    return dtype == DREAM_BF16 && blocks * heads < resident_groups(head_dim) ? MAX_SPLITS : 1;
}

inline size_t compress_most(int batch, int n_heads, int head_dim, int n_q, int vis_len, int dtype)
{
    const int64_t heads = (int64_t)n_heads * batch;
    const int v = vis_len > 0 ? vis_len : 1;
    const size_t lse = most_splits(ceil_div(n_q, BLOCK), heads, head_dim, dtype) * heads * ((n_q + 15) / 16 * 16) * sizeof(float);
    const size_t part = most_splits(ceil_div(v, BLOCK), heads, head_dim, dtype) * heads * v * sizeof(float);
    return DREAM_WORKSPACE_MIN_BYTES + align_up(lse, 256) + align_up(part, 256);
}

}  // namespace dream
