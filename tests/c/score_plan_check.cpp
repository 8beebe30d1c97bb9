// The plans of csrc/score_plan.h for the host: what tests/test_score_plan.py checks.
#include "score_plan.h"

using namespace dream;

static CompressPlan plan;

extern "C" void score_plan(int batch, int heads, int head_dim, int n_q, int n_keys, int vis_start, int vis_len, int with_pos, int entropy, int lse_given, int direct, int *out)
{
    plan = compress_plan(batch, heads, head_dim, n_q, n_keys, vis_start, vis_len, DREAM_BF16, with_pos, entropy, lse_given, direct);
    const int v[] = {plan.ns1, plan.ns2, plan.units1, plan.units2, plan.wide1, plan.wide2, plan.order1.n, plan.order2.n, plan.map1.count[0], plan.map2.count[0]};
    std::copy(std::begin(v), std::end(v), out);
}
// (block by rank, split, splits of the block) of unit u of a pass of the last plan
extern "C" void score_unit(int pass, int u, int *out)
{
    const SplitMap &map = pass == 1 ? plan.map1 : plan.map2;
    const UnitOrder &order = pass == 1 ? plan.order1 : plan.order2;
    const SplitUnit r = split_unit(map, order.n > 0, order.n > 0 ? order.pair[u / 2] : 0, u);
    out[0] = r.rank;
    out[1] = r.split;
    out[2] = r.n;
}
extern "C" long long score_workspace(int batch, int heads, int head_dim, int n_q, int vis_len) { return compress_most(batch, heads, head_dim, n_q, vis_len, DREAM_BF16); }
extern "C" long long score_needs() { return plan.off_part; }
