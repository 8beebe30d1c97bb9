// dream_spec_accept: acceptance over the verified tree at a sampling temperature (Section 2.1: a drafted token
// d is accepted with probability min(1, P_target(d) / P_draft(d)); after a rejection the rest is discarded and
// the target's distribution decides the next token; Section 4 evaluates at temperature 1).  For a tree the
// children of the current node are tried in node order; after a rejected child the target distribution becomes
// the positive part of (target - draft), the rejected token leaves the draft distribution, and the next child is
// tried against those; the first accepted child becomes the current node.  With no accepted child the next
// token is drawn from the current target distribution by inverting its cumulative sum in token order.  The
// uniform random numbers are inputs.
//
// Two launches.  softmax_stats_kernel (parallel over rows and chunks of them) leaves (max, sum of exponentials)
// per chunk for the target and the draft row of every node with children: the only rows a test can need.
// spec_walk_kernel then evaluates the test of every node against its parent's untouched distributions in parallel:
// that is exactly the test the walk performs whenever a node is the first child tried, so the walk descends through
// first children by table lookup.  Where the rows are many the first launch covers the roots only, and the walk works out the statistics of
// a node's two rows when it comes to the node: a handful of nodes per sequence instead of all.
// A rejection needs one number that no table holds, the mass of the new residual
// over the whole vocabulary.  Every residual is a pointwise function of the two logits of a token and of a few
// scalars (the masses of the residuals before it), so it is recomputed from the logit rows and never stored; several
// workgroups share a sequence, each sums its chunks and all exchange one float per chunk.  The masses also give the
// draw, which then reads one chunk.  Every reduction has a fixed order, so the result is reproducible.
// Bound by latency: the exchanges between the workgroups of a sequence follow each other, one per rejection and, with few statistics
// beforehand, one per node.  spec_walk_small_kernel is the walk with that chain cut short; spec_walk_kernel serves what it does not take.
//
// Why several workgroups: one CU pulls 60 to 75 GB/s, 14 us and more for one pass over two float32 rows of 131072 tokens.
// Measured, us per call, four sets of tensors in turn, spec_walk_kernel / spec_walk_small_kernel: 4 sequences x 60 nodes x 131072 float32 logits 46.9 / 28.5, 8 x 60 x 262144 bf16 61.2 / 36.2, 1 x 60 x
// 32000 bf16 31.3 / 23.2; 1 to 1.5 us less where every call has the same tensors.
#include "common.h"
#include <algorithm>
#include <type_traits>

using namespace dream;

namespace {

constexpr int NT = 512;           // threads of the walk
constexpr int NW = NT / 64;

template <bool BF16>
__device__ __forceinline__ float load_logit(const void *p, int64_t i)
{
    return BF16 ? bf16_bits_to_float(reinterpret_cast<const uint16_t *>(p)[i]) : reinterpret_cast<const float *>(p)[i];
}

__device__ __forceinline__ int block_min_int(int v, int *red, int tid)
{
    for (int off = 32; off > 0; off >>= 1)
        v = min(v, __shfl_xor(v, off));
    __syncthreads();
    if ((tid & 63) == 0)
        red[tid >> 6] = v;
    __syncthreads();
    int t = red[0];
#pragma unroll
    for (int w = 1; w < NW; w++)
        t = min(t, red[w]);
    return t;
}

// Logits of a chunk: a workgroup's share of the statistics pass, and what a workgroup of the walk keeps in its registers.  PER groups of 8 a
// thread of the walk: 1, or 2 or 4 where the walk's workgroups would otherwise have several chunks each and read them again in
// every round.
template <int PER>
constexpr int CHUNK = NT * 8 * PER;

// tokens t .. t+7 of a row (t a multiple of 8); `vec`: the row is 16-byte aligned and holds a multiple of 8 tokens.
// Tokens past the end come back as -inf.
template <bool BF16>
__device__ __forceinline__ void load8(const void *base, int64_t row, int t, int vocab, bool vec, float v[8])
{
    if (vec && t + 8 <= vocab) {
        if (BF16) {
            const uint4 u = *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(base) + row + t);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int j = 0; j < 4; j++) {
                v[2 * j] = __uint_as_float(w[j] << 16);
                v[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
            }
        } else {
            const float4 a = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(base) + row + t);
            const float4 c = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(base) + row + t + 4);
            v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = c.x; v[5] = c.y; v[6] = c.z; v[7] = c.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; j++)
            v[j] = t + j < vocab ? load_logit<BF16>(base, row + t + j) : -INFINITY;
    }
}

// The same tokens as they lie in memory, so that they can be asked for long before they are looked at.  VEC stands for `vec`, known when compiling.
template <bool BF16, bool VEC>
struct Raw8 {
    uint4 w[BF16 ? 1 : 2];
    __device__ __forceinline__ void load(const void *base, int64_t row, int t, int vocab)
    {
        if (VEC) {
            const uint32_t none = BF16 ? 0xff80ff80u : 0xff800000u;    // -inf
            w[0] = {none, none, none, none};
            w[BF16 ? 0 : 1] = {none, none, none, none};
            if (t < vocab) {
                const uint4 *p = reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(base) + (row + t) * (BF16 ? 2 : 4));
                w[0] = p[0];
                if (!BF16)
                    w[BF16 ? 0 : 1] = p[1];
            }
        } else {
            uint32_t x[8];
#pragma unroll
            for (int j = 0; j < 8; j++)
                x[j] = __float_as_uint(t + j < vocab ? load_logit<BF16>(base, row + t + j) : -INFINITY);
            if (BF16) {
                w[0] = {x[0] >> 16 | x[1], x[2] >> 16 | x[3], x[4] >> 16 | x[5], x[6] >> 16 | x[7]};
            } else {
                w[0] = {x[0], x[1], x[2], x[3]};
                w[BF16 ? 0 : 1] = {x[4], x[5], x[6], x[7]};
            }
        }
    }
    __device__ __forceinline__ void unpack(float v[8]) const
    {
        const uint4 c = w[BF16 ? 0 : 1];
        const uint32_t x[8] = {w[0].x, w[0].y, w[0].z, w[0].w, c.x, c.y, c.z, c.w};
#pragma unroll
        for (int j = 0; j < 8; j++)
            v[j] = __uint_as_float(!BF16 ? x[j] : j & 1 ? x[j / 2] & 0xffff0000u : x[j / 2] << 16);
    }
};
// A token's exponential times its row's normaliser, and one step of the residual chain.  Written with explicit fused operations, so that
// every loop that evaluates a token (in registers, from memory, at one token) gives it the same bits.
__device__ __forceinline__ float token_mass(float logit, float inv_temp, float m, float inv_z) { return __expf(fmaf(logit, inv_temp, -m)) * inv_z; }
__device__ __forceinline__ float residual(float P, float jp, float Q, float jq) { return fmaxf(fmaf(P, jp, -(Q * jq)), 0.0f); }

// Exchange of the walk's partial sums: slots [B][2][MAX_VAL][MAX_SEG] of (round << 32 | float bits), cleared by
// softmax_stats_kernel, which the stream orders before the walk.
constexpr int MAX_SEG = 64, MAX_VAL = 4;
constexpr int SLOTS = 2 * MAX_VAL * MAX_SEG;
// Units of 64 cycles from publishing to the first poll.  A word takes about 900 cycles to get to the others, and a poll that comes too early holds up the one that would find it.
// spec_walk_small_kernel, 4 sequences x 60 nodes x 131072 float32 logits: first poll at once 36.6 us, after 320 cycles 33.5, 770 30.7, 1020 30.4, 1280 31.1, 1660 32.4.
// spec_walk_kernel, at once / after 900 cycles, by the workgroups of a sequence: 2 73.6 / 75.9, 3 87.1 / 89.9, 4 98.4 / 100.2, 8 88.3 / 88.7 and 46.7 / 47.0, 12 51.2 / 51.2, 13 58.8 / 58.6, 16 54.9 / 54.0,
// 19 59.5 / 57.9, 32 53.5 / 47.7, 64 48.3 / 40.7: from 16 on.
constexpr int POLL_DELAY = 14;

// (max, sum of exp(x/temp - max)) of one chunk of one row of the first n_nodes nodes of a sequence.  z = 0: target rows;
// z = 1: draft rows; nothing for nodes without children (a leaf's target row is summed by the walk if the walk ends there).
template <bool BF16, int PER>
__global__ __launch_bounds__(256) void softmax_stats_kernel(const void *tlogits, const void *dlogits, int n_tree, int n_nodes, int vocab,
                                                            int n_chunks, int vec, const int32_t *parent, float inv_temp, float *stat_m, float *stat_s,
                                                            uint64_t *slots, int64_t rows_all)
{
    const int chunk = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = n_nodes == 1 ? blockIdx.y : blockIdx.y / n_nodes, node = blockIdx.y - b * n_nodes, which = blockIdx.z;
    const int64_t node_row = (int64_t)b * n_tree + node;
    __shared__ float red[4];
    auto clear_slots = [&] {
        if (slots && chunk == 0 && node == 0 && which == 0)
            for (int i = tid; i < SLOTS; i += 256)
                slots[(int64_t)b * SLOTS + i] = 0;
    };
    if (n_nodes > 1) {           // (the root alone is not worth the trip to memory that tells whether it has children)
        clear_slots();
        int kids = 0;
        for (int i = tid; i < n_tree; i += 256)
            kids |= parent[(int64_t)b * n_tree + i] == node;
        if (!__syncthreads_or(kids))
            return;
    }
    const void *base = which ? dlogits : tlogits;
    const int64_t row = node_row * vocab;
    constexpr int STAT_CHUNK = CHUNK<PER>;
    const int begin = chunk * STAT_CHUNK;
    float x[STAT_CHUNK / 256];
    float m = -INFINITY;
    // one question for the whole chunk: with one per group of 8 tokens its load was waited for before the next was asked for (a chunk of 16384 bfloat16 tokens, 32
    // sequences x 8 nodes x 131072: 35.5 us instead of 26.0)
    if (vec && begin + STAT_CHUNK <= vocab) {
#pragma unroll
        for (int r = 0; r < STAT_CHUNK / 2048; r++)
            load8<BF16>(base, row, begin + (r * 256 + tid) * 8, 0x7fffffff, true, x + 8 * r);
    } else {
#pragma unroll
        for (int r = 0; r < STAT_CHUNK / 2048; r++)
            load8<BF16>(base, row, begin + (r * 256 + tid) * 8, vocab, vec, x + 8 * r);
    }
    if (n_nodes == 1)            // (behind the loads: they wait for nothing that way)
        clear_slots();
    const int64_t slot = (which * rows_all + node_row) * n_chunks + chunk;
#pragma unroll
    for (int j = 0; j < STAT_CHUNK / 256; j++) {
        x[j] *= inv_temp;
        m = fmaxf(m, x[j]);
    }
    m = wave_max(m);
    if (lane == 0)
        red[wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    float sum = 0.0f;
    if (m > -INFINITY) {
#pragma unroll
        for (int j = 0; j < STAT_CHUNK / 256; j++)
            sum += __expf(x[j] - m);                          // exp(-inf) = 0 for the padding
    }
    sum = wave_sum(sum);
    __syncthreads();
    if (lane == 0)
        red[wave] = sum;
    __syncthreads();
    if (tid == 0) {
        stat_m[slot] = m;
        stat_s[slot] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}

// (max, sum of exponentials relative to it) of a row from its chunk statistics.  Every lane of a wave calls this: lane
// c takes chunk c (and c + 64, ...), the maximum and then the rescaled sum are reduced with xor shuffles, a fixed order.
__device__ __forceinline__ void merge_row_stats(const float *cm, const float *cs, int n_chunks, int lane, float &m, float &z)
{
    m = -INFINITY;
    for (int c = lane; c < n_chunks; c += 64)
        m = fmaxf(m, cm[c]);
    for (int off = 32; off > 0; off >>= 1)
        m = fmaxf(m, __shfl_xor(m, off));
    z = 0.0f;
    for (int c = lane; c < n_chunks; c += 64) {
        const float s = cs[c];
        if (s > 0.0f)
            z += s * __expf(cm[c] - m);
    }
    for (int off = 32; off > 0; off >>= 1)
        z += __shfl_xor(z, off);
}

struct WalkArgs {
    const void *tlogits, *dlogits;
    int n_tree, vocab, n_chunks;
    int seg_chunks, n_seg;         // a row is n_seg <= MAX_SEG segments of seg_chunks chunks (one chunk up to 1048576 tokens)
    int vec;                       // (whole words: a byte of one is taken from it as soon as the wave starts)
    int lazy;                      // statistics of the roots only; the walk works out those of the nodes it comes to
    const int32_t *token, *parent;
    const float *u_accept, *u_bonus;
    int max_depth;
    float inv_temp;
    int spin_limit;
    const float *stat_m, *stat_s;  // [2][B * n_tree][n_chunks], written for nodes with children
    uint64_t *slots;
    int32_t *accept_len, *accept_path, *bonus_token;
};

// gridDim.x workgroups walk one sequence together.  All of them take every decision (from the same numbers in the same
// order), so they need no commands from each other: in a round each sums its segments (segment s belongs to workgroup
// s % gridDim.x), publishes one word (round, sum) per segment and reads the others'.  The number travels in the word
// itself, so the exchange is relaxed agent-scope loads and stores without fences.  Words of round r + 2 overwrite those
// of round r: nobody publishes round r + 2 before having seen everybody's round r + 1, which everybody publishes after reading round r.
// Nothing depends on the workgroups running at the same time: a wait is bounded, workgroup 0 sums missing segments itself
// (token_mass and residual, added in the same order, so the same bits) and waits for nobody again, any other workgroup that waited in vain ends.
// Only workgroup 0 writes results.
// ALONE: this workgroup sums all segments, whoever else is there.  TREE: nodes there is room for.
template <bool BF16, int PER, bool ALONE, int TREE>
__device__ __forceinline__ void walk(const WalkArgs &a)
{
    __shared__ int32_t s_par[TREE];
    __shared__ int32_t s_tok[TREE];
    __shared__ int32_t s_first[TREE];     // first child of a node, or NONE
    __shared__ float s_mt[TREE], s_zt[TREE];   // target row: max, sum (nodes with children)
    __shared__ float s_md[TREE], s_zd[TREE];   // draft row
    __shared__ float s_px[TREE], s_qx[TREE];   // a node's token at its parent: target and draft exponential
    __shared__ float s_u[TREE];
    __shared__ uint8_t s_ok[TREE];        // the node passes its test when it is the first child tried
    // rejections at the current node: P <- max(P * ip - Q * iq, 0) if `take`, then Q[x] <- 0
    __shared__ float s_ip[TREE], s_iq[TREE];
    __shared__ int32_t s_x[TREE];
    __shared__ uint8_t s_take[TREE];
    __shared__ float s_part[MAX_VAL][MAX_SEG], s_mass[MAX_SEG];
    __shared__ float s_red[2][4][NW], s_scan[NW];
    __shared__ int s_redi[NW];
    constexpr int NONE = 0x7fffffff, STAT_CHUNK = CHUNK<PER>;
    const int b = blockIdx.y, wg = blockIdx.x, n_wg = gridDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_tree = a.n_tree, vocab = a.vocab, n_chunks = a.n_chunks, n_seg = a.n_seg;
    const bool vec = a.vec;
    const float inv_temp = a.inv_temp;
    const int64_t bt = (int64_t)b * n_tree, rows_all = (int64_t)gridDim.y * n_tree;
    const int max_depth = a.max_depth;
    const int n_known = a.lazy ? 1 : n_tree;     // nodes whose statistics the launch before has left
    // Everything a test needs is brought into LDS up front, with as few dependent trips to memory as there are: (parent,
    // token, random number), then (the two logits of every node's token at its parent; the chunk statistics).
    for (int i = tid; i < n_tree; i += NT) {
        int par = a.parent[bt + i];
        const int x = min(max(a.token[bt + i], 0), vocab - 1);   // device metadata is trusted but kept inside the row
        par = par < i ? par : -1;
        s_u[i] = a.u_accept[bt + i];
        s_par[i] = par;
        s_tok[i] = x;
        s_first[i] = NONE;
        if (i > 0 && par >= 0) {
            s_px[i] = load_logit<BF16>(a.tlogits, (bt + par) * vocab + x) * inv_temp;
            s_qx[i] = load_logit<BF16>(a.dlogits, (bt + par) * vocab + x) * inv_temp;
        }
    }
    int32_t *path = a.accept_path + (int64_t)b * (max_depth + 1);
    if (wg == 0)
        for (int i = tid; i <= max_depth; i += NT)
            path[i] = i == 0 ? 0 : -1;
    __syncthreads();
    for (int i = tid; i < n_tree; i += NT)
        if (i > 0 && s_par[i] >= 0)
            atomicMin(&s_first[s_par[i]], i);
    __syncthreads();
    if (n_chunks <= 64) {
        // a node per pass of a wave, a chunk per lane; four nodes' loads in flight
        for (int i0 = wave * 4; i0 < n_known; i0 += NW * 4) {
            float m[4][2], z[4][2];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const bool live = i0 + u < n_known && lane < n_chunks && s_first[min(i0 + u, n_tree - 1)] != NONE;
#pragma unroll
                for (int w = 0; w < 2; w++) {
                    const int64_t at = live ? (w * rows_all + bt + i0 + u) * n_chunks + lane : 0;
                    m[u][w] = live ? a.stat_m[at] : -INFINITY;
                    z[u][w] = live ? a.stat_s[at] : 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; u++)
#pragma unroll
                for (int w = 0; w < 2; w++) {
                    const float mx = wave_max(m[u][w]);
                    const float sum = wave_sum(z[u][w] > 0.0f ? z[u][w] * __expf(m[u][w] - mx) : 0.0f);
                    if (lane == 0 && i0 + u < n_known && s_first[i0 + u] != NONE) {
                        (w ? s_md : s_mt)[i0 + u] = mx;
                        (w ? s_zd : s_zt)[i0 + u] = sum;
                    }
                }
        }
    } else {
        for (int i = wave; i < n_known; i += NW) {
            if (s_first[i] == NONE)
                continue;
            float mt, zt, md, zd;
            merge_row_stats(a.stat_m + (bt + i) * n_chunks, a.stat_s + (bt + i) * n_chunks, n_chunks, lane, mt, zt);
            merge_row_stats(a.stat_m + (rows_all + bt + i) * n_chunks, a.stat_s + (rows_all + bt + i) * n_chunks, n_chunks, lane, md, zd);
            if (lane == 0) {
                s_mt[i] = mt; s_zt[i] = zt; s_md[i] = md; s_zd[i] = zd;
            }
        }
    }
    __syncthreads();
    // the test every child of nodes first .. last faces when it is the first one tried
    auto test_children = [&](int first, int last) {
        for (int i = tid; i < n_tree; i += NT) {
            const int p = s_par[i];
            if (i > 0 && p >= first && p <= last) {
                const float px = s_px[i] = __expf(s_px[i] - s_mt[p]);
                const float qx = s_qx[i] = __expf(s_qx[i] - s_md[p]);
                const float ratio = qx > 0.0f ? (px / s_zt[p]) / (qx / s_zd[p]) : (px > 0.0f ? INFINITY : 0.0f);
                s_ok[i] = s_u[i] < fminf(1.0f, ratio);
            }
        }
    };
    test_children(0, n_known - 1);
    __syncthreads();

    auto next_sibling = [&](int node) {      // every wave finds it for itself: no barrier
        for (int i0 = node & ~63; i0 < n_tree; i0 += 64) {
            const int i = i0 + lane;
            const uint64_t hit = __ballot(i > node && i < n_tree && s_par[min(i, n_tree - 1)] == s_par[node]);
            if (hit)
                return i0 + __builtin_ctzll(hit);
        }
        return NONE;
    };

    int cur = 0, depth = 0, n_rej = 0;
    int64_t row = bt * vocab;                               // of the current node
    float mt = 0.0f, md = 0.0f, ip = 0.0f, iq = 0.0f;       // its rows' normalisers: p = exp(t - mt) * ip, q = exp(d - md) * iq
    // residual target and reduced draft of token t after the first n rejections at the current node
    auto chain = [&](int n, int t, float &P, float &Q) {
        for (int j = 0; j < n; j++) {
            const float r = residual(P, s_ip[j], Q, s_iq[j]);
            P = s_take[j] ? r : P;
            Q = t == s_x[j] ? 0.0f : Q;
        }
    };
    auto fetch_residual = [&](int n, int t, float v[8]) {
        float dv[8];
        load8<BF16>(a.tlogits, row, t, vocab, vec, v);
        load8<BF16>(a.dlogits, row, t, vocab, vec, dv);
#pragma unroll
        for (int j = 0; j < 8; j++) {
            v[j] = token_mass(v[j], inv_temp, mt, ip);      // (0 past the end: the logits read as -inf there)
            dv[j] = token_mass(dv[j], inv_temp, md, iq);
        }
        for (int i = 0; i < n; i++) {
            const float jp = s_ip[i], jq = s_iq[i];
            const bool take = s_take[i];
            const int x = s_x[i] - t;
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const float r = residual(v[j], jp, dv[j], jq);
                v[j] = take ? r : v[j];
                dv[j] = x == j ? 0.0f : dv[j];
            }
        }
    };
    // A workgroup with one chunk keeps its residual target and reduced draft in registers from round to round: rp, rq hold
    // them after the first reg_n rejections at the current node (RAW: the logits; UNREAD: nothing yet).
    constexpr int RAW = -1, UNREAD = -2;
    float rp[PER][8], rq[PER][8];
    int reg_n = UNREAD;
    const bool keeps = n_seg <= n_wg && a.seg_chunks == 1;
    auto read_own = [&]() {
#pragma unroll
        for (int h = 0; h < PER; h++) {
            load8<BF16>(a.tlogits, row, wg * STAT_CHUNK + (h * NT + tid) * 8, vocab, vec, rp[h]);
            load8<BF16>(a.dlogits, row, wg * STAT_CHUNK + (h * NT + tid) * 8, vocab, vec, rq[h]);
        }
        reg_n = RAW;
    };
    // The waves' values meet in one of two places in turn: whoever writes a place again has passed the barrier behind the reads of it.
    int red_at = 0;
    auto block_sum = [&](float v) {
        float *red = s_red[red_at][0];
        red_at ^= 1;
        v = wave_sum(v);
        if (lane == 0)
            red[wave] = v;
        __syncthreads();
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; w++)
            t += red[w];
        return t;
    };
    // (max, sum of exponentials) of a chunk of a target row, its logits in x, and with `two` of a draft row, joined to those of the chunks
    // before it: every wave relative to its own maximum, then the waves in order
    auto add_stats = [&](const float (&x)[PER][8], const float (&y)[PER][8], bool two, float (&val)[MAX_VAL]) {
        float(&red)[4][NW] = s_red[red_at];
        red_at ^= 1;
        auto of_wave = [&](const float (&r)[PER][8], int at) {
            float mx = -INFINITY, sum = 0.0f;
#pragma unroll
            for (int h = 0; h < PER; h++)
#pragma unroll
                for (int j = 0; j < 8; j++)
                    mx = fmaxf(mx, r[h][j] * inv_temp);
            mx = wave_max(mx);
            const float ms = mx == -INFINITY ? 0.0f : mx;
#pragma unroll
            for (int h = 0; h < PER; h++)
#pragma unroll
                for (int j = 0; j < 8; j++)
                    sum += __expf(r[h][j] * inv_temp - ms);       // (0 for the padding)
            sum = wave_sum(sum);
            if (lane == 0) {
                red[at][wave] = mx;
                red[at + 1][wave] = sum;
            }
        };
        of_wave(x, 0);
        if (two)
            of_wave(y, 2);
        __syncthreads();
        auto join = [&](int at) {
            float m = val[at], z;
#pragma unroll
            for (int w = 0; w < NW; w++)
                m = fmaxf(m, red[at][w]);
            z = val[at + 1] > 0.0f ? val[at + 1] * __expf(val[at] - m) : 0.0f;
#pragma unroll
            for (int w = 0; w < NW; w++)
                z += red[at + 1][w] > 0.0f ? red[at + 1][w] * __expf(red[at][w] - m) : 0.0f;
            val[at] = m;
            val[at + 1] = z;
        };
        join(0);
        if (two)
            join(2);
    };
    // A segment's share of a round: the mass of the residual after n rejections (n > 0), (max, sum of exponentials) of the target row
    // (TARGET), or those of the target row and of the draft row (BOTH).
    constexpr int TARGET = 0, BOTH = -1;
    auto values_of = [&](int n) { return n > 0 ? 1 : n == TARGET ? 2 : 4; };
    auto segment = [&](int seg, int n, float (&val)[MAX_VAL]) {
        val[0] = val[2] = n > 0 ? 0.0f : -INFINITY;
        val[1] = val[3] = 0.0f;
        if (n != TARGET && keeps && seg == wg) {
            if (reg_n == UNREAD)
                read_own();
            if (n == BOTH) {
                add_stats(rp, rq, true, val);
                return;
            }
            if (reg_n == RAW) {
#pragma unroll
                for (int h = 0; h < PER; h++)
#pragma unroll
                    for (int j = 0; j < 8; j++) {
                        rp[h][j] = token_mass(rp[h][j], inv_temp, mt, ip);
                        rq[h][j] = token_mass(rq[h][j], inv_temp, md, iq);
                    }
                reg_n = 0;
            }
            for (; reg_n < n - 1; reg_n++) {     // steps whose outcome is known
                const float jp = s_ip[reg_n], jq = s_iq[reg_n];
                const bool take = s_take[reg_n];
                const int x = s_x[reg_n] - seg * STAT_CHUNK - tid * 8;
#pragma unroll
                for (int h = 0; h < PER; h++)
#pragma unroll
                    for (int j = 0; j < 8; j++) {
                        const float r = residual(rp[h][j], jp, rq[h][j], jq);
                        rp[h][j] = take ? r : rp[h][j];
                        rq[h][j] = x == h * NT * 8 + j ? 0.0f : rq[h][j];
                    }
            }
            const float jp = s_ip[n - 1], jq = s_iq[n - 1];   // the last one is only summed: whether it is taken depends on the sum
            float s = 0.0f;
#pragma unroll
            for (int h = 0; h < PER; h++)
#pragma unroll
                for (int j = 0; j < 8; j++)
                    s += residual(rp[h][j], jp, rq[h][j], jq);
            val[0] = block_sum(s);
            return;
        }
        for (int c = seg * a.seg_chunks; c < min((seg + 1) * a.seg_chunks, n_chunks); c++) {
            float v[PER][8];
            const int t = c * STAT_CHUNK + tid * 8;
            if (n > 0) {
                float s = 0.0f;
#pragma unroll
                for (int h = 0; h < PER; h++)
                    fetch_residual(n, t + h * NT * 8, v[h]);
#pragma unroll
                for (int h = 0; h < PER; h++)
#pragma unroll
                    for (int j = 0; j < 8; j++)
                        s += v[h][j];
                val[0] += block_sum(s);
            } else {
                float d[PER][8];
#pragma unroll
                for (int h = 0; h < PER; h++) {
                    load8<BF16>(a.tlogits, row, t + h * NT * 8, vocab, vec, v[h]);
                    if (n == BOTH)
                        load8<BF16>(a.dlogits, row, t + h * NT * 8, vocab, vec, d[h]);
                }
                add_stats(v, d, n == BOTH, val);
            }
        }
    };
    auto sum_segments = [&](const float *v) {     // every lane of every wave: the same tree over the segments
        return wave_sum(lane < n_seg ? v[lane] : 0.0f);
    };
    int round = 0;
    bool alone = ALONE || n_wg == 1;
    // One round: fills s_part for all segments.  False: this workgroup waited in vain and ends.
    auto exchange = [&](int n) {
        round++;
        uint64_t *slot = a.slots + (int64_t)b * SLOTS + (round & 1) * MAX_VAL * MAX_SEG;
        const int n_val = values_of(n);
        for (bool again = false;; again = true) {           // (again: the segments that others did not sum)
            for (int seg = alone || again ? 0 : wg; seg < n_seg; seg += alone || again ? 1 : n_wg) {
                if (again && seg % n_wg == wg)
                    continue;
                float val[MAX_VAL];
                segment(seg, n, val);
                if (tid < n_val) {
                    const float v = tid == 0 ? val[0] : tid == 1 ? val[1] : tid == 2 ? val[2] : val[3];
                    s_part[tid][seg] = v;
                    if (!alone && !again)
                        __hip_atomic_store(slot + tid * MAX_SEG + seg, ((uint64_t)(uint32_t)round << 32) | __float_as_uint(v), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if (again)
                alone = true;
            if (alone)
                break;
            bool missing = false;
            const int val = tid / MAX_SEG, seg = tid % MAX_SEG;
            if (n_wg >= 16)              // fewer workgroups do not hold each other up
                __builtin_amdgcn_s_sleep(POLL_DELAY);
            if (val < n_val && seg < n_seg && seg % n_wg != wg) {
                uint64_t w = 0;
                missing = true;
                for (int spin = 0; spin < a.spin_limit && missing; spin++) {
                    w = __hip_atomic_load(slot + val * MAX_SEG + seg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    missing = (uint32_t)(w >> 32) != (uint32_t)round;
                    if (missing)
                        __builtin_amdgcn_s_sleep(1);
                }
                if (!missing)
                    s_part[val][seg] = __uint_as_float((uint32_t)w);
            }
            if (!__syncthreads_or(missing))
                break;
            if (wg != 0)
                return false;
        }
        __syncthreads();
        return true;
    };

    // Inverse-CDF draw over the values of tokens [r0, r1) (r0 a multiple of 8), read through `fetch8(t, v)` (8 tokens
    // from t, zeros past the vocabulary): `mass_before` is the mass below r0, `target` the point to invert.  Contiguous
    // tokens per thread, block scan, the owning thread rescans.  Without an owner (rounding left the target at or above
    // the sum) the last token with mass in the range is taken.
    auto draw = [&](int r0, int r1, float mass_before, float target, auto fetch8) {
        const int cpt = (((r1 - r0) + NT - 1) / NT + 7) & ~7;
        const int t0 = min(r0 + tid * cpt, r1), t1 = min(t0 + cpt, r1);
        float local = 0.0f;
        for (int t = t0; t < t1; t += 8) {
            float v[8];
            fetch8(t, v);
#pragma unroll
            for (int j = 0; j < 8; j++)
                local += v[j];
        }
        float inc = local;   // inclusive scan of the per-thread sums: inside a wave by shuffles, wave totals through LDS
        for (int off = 1; off < 64; off <<= 1) {
            const float o = __shfl_up(inc, off);
            if (lane >= off)
                inc += o;
        }
        __syncthreads();
        if (lane == 63)
            s_scan[wave] = inc;
        __syncthreads();
        float base = mass_before;
#pragma unroll
        for (int w = 0; w < NW; w++)
            if (w < wave)
                base += s_scan[w];
        const float before = base + inc - local;        // mass of all tokens below t0
        int owner = (before + local > target && t1 > t0) ? tid : NONE;
        owner = block_min_int(owner, s_redi, tid);
        if (owner == NONE) {
            int last = -1;
            for (int t = t0; t < t1; t += 8) {
                float v[8];
                fetch8(t, v);
#pragma unroll
                for (int j = 0; j < 8; j++)
                    if (v[j] > 0.0f)
                        last = t + j;
            }
            last = -block_min_int(-last, s_redi, tid);
            if (tid == 0)
                a.bonus_token[b] = last >= 0 ? last : min(r0, vocab - 1);
        } else if (tid == owner) {
            float run = before;
            int pick = t1 - 1;
            bool found = false;
            for (int t = t0; t < t1 && !found; t += 8) {
                float v[8];
                fetch8(t, v);
#pragma unroll
                for (int j = 0; j < 8; j++) {
                    run += v[j];
                    if (!found && run > target && t + j < t1) {
                        pick = t + j;
                        found = true;
                    }
                }
            }
            a.bonus_token[b] = pick;
        }
    };
    // The draw when s_mass holds the mass of every segment: the segment with the drawn point is found from those sums,
    // in order, and only that one is read.
    auto draw_by_segments = [&](auto fetch8) {
        const float mine = lane < n_seg ? s_mass[lane] : 0.0f;
        float upto = mine;                      // of the segments up to lane's
        for (int off = 1; off < 64; off <<= 1) {
            const float o = __shfl_up(upto, off);
            if (lane >= off)
                upto += o;
        }
        const float prev = __shfl_up(upto, 1), below = lane ? prev : 0.0f;
        const float target = a.u_bonus[b] * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(upto), 63));
        const uint64_t past = __ballot(mine > 0.0f && upto > target), some = __ballot(mine > 0.0f);
        // (rounding may leave the target at or above the total: the last segment with mass)
        const int pick = past ? __builtin_ctzll(past) : some ? 63 - __builtin_clzll(some) : 0;
        const float before = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(below), pick));
        const int64_t seg_tokens = (int64_t)a.seg_chunks * STAT_CHUNK;
        draw((int)(pick * seg_tokens), (int)min((pick + 1) * seg_tokens, (int64_t)vocab), before, target, fetch8);
    };

    bool have_mass = false;                    // s_mass holds the masses of the segments of the current target
    int first = NONE, child = NONE;
    float Zp = 1.0f, Zq = 1.0f, qx = 0.0f;     // masses of the current P and Q; the rejected child's draft probability
    // `child` is rejected: the target becomes the positive part of (target - draft), its token leaves the draft
    auto reject = [&]() {
        const int x = s_tok[child];
        if (tid == 0) {
            s_ip[n_rej] = 1.0f / Zp;
            s_iq[n_rej] = Zq > 0.0f ? 1.0f / Zq : 0.0f;
            s_x[n_rej] = x;
            s_take[n_rej] = 1;
        }
        __syncthreads();
        qx = s_qx[child] * iq;
        for (int j = 0; j < n_rej; j++)
            qx = s_x[j] == x ? 0.0f : qx;
    };
    auto visit = [&](int node) {
        cur = node;
        depth++;
        if (wg == 0 && tid == 0)
            path[depth] = cur;
        row = (bt + cur) * vocab;
        have_mass = false;
        reg_n = UNREAD;
    };
    // `ask` is what the next round is about: BOTH, TARGET, the number of rejections with the last one, or nothing before the walk has gone
    // down from the current node (DESCEND).  (All workgroups of the sequence go the same way.)
    constexpr int DESCEND = -2;
    for (int ask = DESCEND;;) {
        if (ask == DESCEND) {
            // ---- through first children whose (precomputed) test passes
            first = depth < max_depth ? s_first[cur] : NONE;
            bool learn = false;
            while (first != NONE && s_ok[first] && !learn) {
                visit(first);
                first = depth < max_depth ? s_first[cur] : NONE;
                learn = a.lazy && s_first[cur] != NONE;
            }
            n_rej = 0;
            if (learn) {
                ask = BOTH;
            } else if (s_first[cur] != NONE) {              // (a node at the depth limit may have children)
                mt = s_mt[cur];
                md = s_md[cur];
                ip = 1.0f / s_zt[cur];
                iq = s_zd[cur] > 0.0f ? 1.0f / s_zd[cur] : 0.0f;
                Zp = Zq = 1.0f;
                child = first;
                if (child == NONE)
                    break;
                reject();
                ask = 1;
            } else {
                ask = TARGET;
            }
        }
        if (!exchange(ask))
            return;
        if (ask == BOTH) {
            // ---- the statistics of the current node's rows, and with them the tests of its children; the masses of its target's segments
            float m[2], z[2];
#pragma unroll
            for (int w = 0; w < 2; w++) {      // lane s: segment s; the same tree over the segments in every wave
                const float ms = lane < n_seg ? s_part[2 * w][lane] : -INFINITY, zs = lane < n_seg ? s_part[2 * w + 1][lane] : 0.0f;
                m[w] = wave_max(ms);
                z[w] = wave_sum(zs > 0.0f ? zs * __expf(ms - m[w]) : 0.0f);
            }
            if (tid < n_seg)
                s_mass[tid] = s_part[1][tid] > 0.0f ? s_part[1][tid] * __expf(s_part[0][tid] - m[0]) * (1.0f / z[0]) : 0.0f;
            if (tid == 0) {
                s_mt[cur] = m[0]; s_zt[cur] = z[0]; s_md[cur] = m[1]; s_zd[cur] = z[1];
            }
            have_mass = true;
            __syncthreads();
            test_children(cur, cur);
            __syncthreads();
            ask = DESCEND;
            continue;
        }
        if (ask == TARGET) {
            mt = wave_max(lane < n_seg ? s_part[0][lane] : -INFINITY);
            ip = 1.0f;
            if (tid < n_seg)
                s_mass[tid] = s_part[1][tid] > 0.0f ? s_part[1][tid] * __expf(s_part[0][tid] - mt) : 0.0f;
            have_mass = true;
            break;
        }
        // ---- `child` is rejected: the mass of what is left of the target
        const float Z = sum_segments(s_part[0]);
        if (Z > 0.0f) {
            Zp = Z;
            have_mass = true;
            if (tid < n_seg)
                s_mass[tid] = s_part[0][tid];
        } else if (tid == 0) {
            s_take[n_rej] = 0;                               // target == draft: the residual is empty and the target stays as it is
        }
        Zq = fmaxf(Zq - qx, 0.0f);
        n_rej++;
        __syncthreads();
        child = next_sibling(child);
        if (child == NONE)
            break;
        float P = s_px[child] * ip, Q = s_qx[child] * iq;
        chain(n_rej, s_tok[child], P, Q);
        const float ratio = Q > 0.0f ? (P / Zp) / (Q / Zq) : (P > 0.0f ? INFINITY : 0.0f);
        if (s_u[child] < fminf(1.0f, ratio)) {
            visit(child);
            __syncthreads();   // the lists of the node before are rewritten: finish reading them first
            ask = a.lazy && s_first[cur] != NONE ? BOTH : DESCEND;
            n_rej = 0;
        } else {
            reject();
            ask = n_rej + 1;
        }
    }
    // ---- no child, or every child rejected: draw from the current target
    if (wg != 0)
        return;
    if (!have_mass && tid < n_seg) {                         // the untouched target
        float s = 0.0f;
        for (int c = tid * a.seg_chunks; c < min((tid + 1) * a.seg_chunks, n_chunks); c++) {
            const float sc = a.stat_s[(bt + cur) * n_chunks + c];
            s += sc > 0.0f ? sc * __expf(a.stat_m[(bt + cur) * n_chunks + c] - mt) : 0.0f;
        }
        s_mass[tid] = s * ip;
    }
    __syncthreads();
    if (n_rej)
        draw_by_segments([&](int t, float v[8]) { fetch_residual(n_rej, t, v); });
    else
        draw_by_segments([&](int t, float v[8]) {
            load8<BF16>(a.tlogits, row, t, vocab, vec, v);
#pragma unroll
            for (int j = 0; j < 8; j++)
                v[j] = token_mass(v[j], inv_temp, mt, ip);
        });
    if (tid == 0)
        a.accept_len[b] = depth;
}

template <bool BF16, int PER>
__global__ __launch_bounds__(NT) void spec_walk_kernel(WalkArgs a)
{
    walk<BF16, PER, false, DREAM_MAX_TREE_ACCEPT>(a);
}

// The walk of a tree of up to 64 nodes whose segments have a workgroup each and are one chunk: what serving asks for.  The same rounds, exchange and
// arithmetic as above, but a round is a chain of trips to memory and LDS and of dependent instructions, so here it has two barriers and what can be had beforehand is:
// - NW waves hold the tokens; one more, the messenger, adds their sums behind the first barrier, publishes and polls, and hands out everybody's sums at the second.
// - Lane i of every wave holds node i: parent, token, random number, the logits of its token at its parent, and what the rejections so far have left of target and draft
//   there.  Each wave takes every decision by itself, in registers.
// - While a round is on its way, the waves work out all of the next step that does not need its sum, and ask for the rows of the node that comes next if the
//   test passes which the round decides.
// A workgroup that waits in vain ends, workgroup 0 then starts over with the walk above, alone.
// us per rejection / visited node with statistics to work out, walk above 3.3 / 4.9, here 1.8 / 3.0.  A call, both, four sets of tensors in turn: 4 sequences x 60 nodes x 131072 float32 logits 46.9 / 28.5,
// 4 x 60 x 262144 bf16 56.3 / 28.8, 32 x 60 x 32000 bf16 49.8 / 30.0, 1 x 60 x 32000 bf16 31.3 / 23.2, 16 x 60 x 131072 bf16 59.7 / 37.4.  (Workgroups of a sequence on one XCD: 40.6
// instead of 37.5 before the first poll was put off.)
template <bool BF16, int PER, bool VEC>
__global__ __launch_bounds__(NT + 64) void spec_walk_small_kernel(const int32_t *parent, const int32_t *token, const float *u_accept, const float *u_draw, const void *tlogits, const void *dlogits,
                                                                  int tree_nodes, int tokens, WalkArgs rest)
{
    // (Plain arguments: in scalar registers when a wave starts, so the first loads wait for nothing; all others are asked for at once.  With them in memory, the random numbers behind the
    // tokens, and what softmax_stats_kernel reads behind what it clears, 4 sequences x 60 nodes x 131072 float32 25.1 to 25.8 us, 23.8 to 24.4 so.)
    WalkArgs a = rest;
    a.parent = parent; a.token = token; a.u_accept = u_accept; a.u_bonus = u_draw; a.tlogits = tlogits; a.dlogits = dlogits; a.n_tree = tree_nodes; a.vocab = tokens;
    __shared__ float s_part[2][MAX_VAL][MAX_SEG];
    __shared__ __attribute__((aligned(16))) float s_red[2][MAX_VAL][NW];
    __shared__ int s_missing[2];
    __shared__ float s_stat[4][64], s_logit[2][64];
    struct alignas(16) Step {
        float jp, jq;
        int32_t x, take;
    };
    __shared__ Step s_step[64];
    __shared__ float s_scan[NW];
    __shared__ int s_redi[NW], s_last[NW];
    constexpr int PIECES = BF16 ? 1 : 2, ROW_BYTES = NT * 16 * PIECES * PER;      // 16-byte pieces of 8 tokens; bytes of a workgroup's tokens
    constexpr bool AHEAD = VEC && ROW_BYTES <= 16384;       // (up to 8 MB a round; workgroups with more to read are bound by that)
    __shared__ __attribute__((aligned(16))) unsigned char s_rows[AHEAD ? 4 * ROW_BYTES : 16];   // target and draft row of the root, and of the node asked for ahead
    const int b = blockIdx.y, wg = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool messenger = wave == NW;
    const int n_tree = a.n_tree, vocab = a.vocab, n_seg = a.n_seg, max_depth = a.max_depth;
    const float inv_temp = a.inv_temp;
    const int64_t bt = (int64_t)b * n_tree;
    using Row = Raw8<BF16, VEC>;
    const int t_own = (wg * PER * NT + tid) * 8;            // this thread's tokens: 8 from here on, and from every NT * 8 behind
    auto of_lane = [](float x, int i) __attribute__((always_inline)) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), i)); };

    // ---- (parent, token, random number), then (the logits of every node's token at its parent; the statistics there are)
    int cur = 0, depth = 0, n_rej = 0;
    // Rows asked for ahead go straight to LDS, each wave's to where it reads them: as values in registers the compiler waits for them at the next branch.
    const uint32_t lds_rows = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)s_rows;
    auto ask_row = [&](const void *logits, int n, int at) __attribute__((always_inline)) {
        const char *base = reinterpret_cast<const char *>(logits) + (bt + n) * vocab * (BF16 ? 2 : 4);
#pragma unroll
        for (int i = 0; i < PER * PIECES; i++) {
            const int t = t_own + i / PIECES * (NT * 8);
            if (AHEAD && t < vocab)
                lds_load16(base, (uint32_t)t * (BF16 ? 2 : 4) + i % PIECES * 16, __builtin_amdgcn_readfirstlane(lds_rows + at * ROW_BYTES + (wave * PER * PIECES + i) * 1024));
        }
    };
    auto asked_row = [&](int at, float(&v)[PER][8]) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < PER; h++) {
            Row r;
#pragma unroll
            for (int i = 0; i < PIECES; i++)
                r.w[i] = *reinterpret_cast<const uint4 *>(s_rows + at * ROW_BYTES + (wave * PER * PIECES + h * PIECES + i) * 1024 + lane * 16);
            r.unpack(v[h]);
#pragma unroll
            for (int j = 0; j < 8; j++)
                v[h][j] = t_own + h * (NT * 8) < vocab ? v[h][j] : -INFINITY;
        }
    };
    auto read_row = [&](const void *logits, float(&v)[PER][8]) __attribute__((always_inline)) {
        Row r[PER];
#pragma unroll
        for (int h = 0; h < PER; h++)
            r[h].load(logits, (bt + cur) * vocab, t_own + h * (NT * 8), vocab);
#pragma unroll
        for (int h = 0; h < PER; h++)
            r[h].unpack(v[h]);
    };
    const bool node = lane < n_tree;
    // (all asked for at once: a load under a condition is waited for where the condition ends)
    const int64_t own = bt + min(lane, n_tree - 1);
    const int par_own = a.parent[own], tok_own = a.token[own];
    const float u_own = a.u_accept[own], u_bonus = a.u_bonus[b];
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::"s"(u_bonus), "s"(a.n_seg), "s"(a.max_depth), "s"(a.inv_temp), "s"(a.spin_limit), "s"(a.stat_m), "s"(a.stat_s), "s"(a.slots), "s"(a.accept_len), "s"(a.accept_path),
                 "s"(a.bonus_token));
    int par_l = node ? par_own : -1;
    const int tok_l = node ? min(max(tok_own, 0), vocab - 1) : 0;                // device metadata is trusted but kept inside the row
    const float u_l = node ? u_own : 0.0f;
    par_l = lane > 0 && par_l >= 0 && par_l < lane ? par_l : -1;
    uint64_t kids = __ballot(par_l == 0);                   // children of the current node that have not been tried
    int asked = -1;                                         // the node whose rows were asked for last (where AHEAD)
    auto ask_rows = [&](int n) __attribute__((always_inline)) {
        if (!AHEAD)
            return;
        asked = n;
        ask_row(a.tlogits, n, 2);
        if (__ballot(par_l == n))                           // (of a leaf only the target is needed)
            ask_row(a.dlogits, n, 3);
    };
    // (a wave waits for its loads in order: those of the messenger are the ones that the first test needs)
    const int64_t rows_all = (int64_t)gridDim.y * n_tree;
    float m[2], z[2];
    auto load_stats = [&](int n) __attribute__((always_inline)) {
#pragma unroll
        for (int w = 0; w < 2; w++) {
            const int64_t at = (w * rows_all + bt + n) * n_seg + lane;
            m[w] = lane < n_seg ? a.stat_m[at] : -INFINITY;
            z[w] = lane < n_seg ? a.stat_s[at] : 0.0f;
        }
    };
    auto store_stats = [&](int n) __attribute__((always_inline)) {
#pragma unroll
        for (int w = 0; w < 2; w++) {
            const float mx = wave_max(m[w]), sum = wave_sum(z[w] > 0.0f ? z[w] * __expf(m[w] - mx) : 0.0f);
            if (lane == 0) {
                s_stat[2 * w][n] = mx;
                s_stat[2 * w + 1][n] = sum;
            }
        }
    };
    if (messenger) {
        float t = 0.0f, d = 0.0f;
        if (par_l >= 0) {
            t = load_logit<BF16>(a.tlogits, (bt + par_l) * vocab + tok_l);
            d = load_logit<BF16>(a.dlogits, (bt + par_l) * vocab + tok_l);
        }
        if (a.lazy)
            load_stats(0);
        s_logit[0][lane] = t * inv_temp;
        s_logit[1][lane] = d * inv_temp;
        if (a.lazy)
            store_stats(0);
        int32_t *path = a.accept_path + (int64_t)b * (max_depth + 1);
        if (wg == 0)
            for (int i = lane; i <= max_depth; i += 64)
                path[i] = i == 0 ? 0 : -1;
    } else {
        if (!a.lazy)                                        // (what a node without children has there is of no use, and not used)
            for (int i = wave; i < n_tree; i += NW) {
                load_stats(i);
                store_stats(i);
            }
        ask_row(a.tlogits, 0, 0);
        if (kids)
            ask_row(a.dlogits, 0, 1);
        if (kids && max_depth > 0)
            ask_rows(__builtin_ctzll(kids));
    }
    __syncthreads();
    const float tx_l = s_logit[0][lane], dx_l = s_logit[1][lane];
    const float mt_l = s_stat[0][lane], zt_l = s_stat[1][lane], md_l = s_stat[2][lane], zd_l = s_stat[3][lane];

    float rp[PER][8], rq[PER][8];                           // this thread's residual target and reduced draft at the current node
    float mt = of_lane(mt_l, 0), zt = of_lane(zt_l, 0), md = of_lane(md_l, 0), zd = of_lane(zd_l, 0);   // of its rows
    float ip = 0.0f, iq = 0.0f;                             // normalisers: p = exp(t - mt) * ip, q = exp(d - md) * iq
    float mass_l = 0.0f;                                    // of segment `lane` of the current target,
    bool have_mass = false;                                 // if this is set
    float left_l = 0.0f;
    // the current node's logits
    auto read_own = [&](bool draft) __attribute__((always_inline)) {
        if (AHEAD && (cur == 0 || asked == cur)) {
            const int at = cur == 0 ? 0 : 2;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            asked_row(at, rp);
            if (draft)
                asked_row(at + 1, rq);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (before others are asked for)
        } else {
            read_row(a.tlogits, rp);
            if (draft)
                read_row(a.dlogits, rq);
        }
    };
    // (max, sum of exponentials) of this wave's share of a row
    auto wave_stats = [&](const float(&x)[PER][8], float &m, float &z) __attribute__((always_inline)) {
        float mx = -INFINITY, sum = 0.0f;
#pragma unroll
        for (int i = 0; i < PER * 8; i++)
            mx = fmaxf(mx, x[i / 8][i % 8] * inv_temp);
        mx = wave_max(mx);
        const float ms = mx == -INFINITY ? 0.0f : mx;
#pragma unroll
        for (int i = 0; i < PER * 8; i++)
            sum += __expf(x[i / 8][i % 8] * inv_temp - ms);  // (0 for the padding)
        m = mx;
        z = wave_sum(sum);
    };
    uint32_t round = 0;
    // The waves' values of a round are in s_red[round & 1]; behind this all segments' are in s_part[round & 1].  V: 1 the mass of a residual, 2 and 4 (max, sum
    // of exponentials) of the target, and of the draft.  `then`: what else the waves that hold tokens have to do.
    auto exchange = [&](auto values, auto then) __attribute__((always_inline)) {
        constexpr int V = decltype(values)::value;
        const int at = round & 1;
        __syncthreads();
        if (messenger) {
            float mine;                                     // value `lane`
            if (V == 1) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(&s_red[at][0][0]), y = *reinterpret_cast<const f32x4 *>(&s_red[at][0][4]);
                mine = ((((((x[0] + x[1]) + x[2]) + x[3]) + y[0]) + y[1]) + y[2]) + y[3];
            } else {
                const int w = lane >> 4 & 1, i = lane & 15;      // a row of 16 lanes: the target's waves, the next one: the draft's
                const bool has = lane < 16 * (V / 2) && i < NW;
                const float m = has ? s_red[at][2 * w][i & (NW - 1)] : -INFINITY, z = has ? s_red[at][2 * w + 1][i & (NW - 1)] : 0.0f;
                const float mx = row_max(m), e = z > 0.0f ? z * __expf(m - mx) : 0.0f;
                float sum[2] = {0.0f, 0.0f};
#pragma unroll
                for (int v = 0; v < V / 2; v++)
#pragma unroll
                    for (int k = 0; k < NW; k++)
                        sum[v] += of_lane(e, 16 * v + k);
                const float m0 = of_lane(mx, 0), m1 = of_lane(mx, 16);
                mine = lane == 0 ? m0 : lane == 1 ? sum[0] : lane == 2 ? m1 : sum[1];
            }
            uint64_t *slot = a.slots + (int64_t)b * SLOTS + at * MAX_VAL * MAX_SEG;
            if (lane < V) {
                s_part[at][lane][wg] = mine;
                if (n_seg > 1)
                    __hip_atomic_store(slot + lane * MAX_SEG + wg, ((uint64_t)round << 32) | __float_as_uint(mine), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            const bool theirs = lane < n_seg && lane != wg;
            bool missing = theirs;
            uint64_t w[V];
            __builtin_amdgcn_s_sleep(POLL_DELAY);
            if (theirs)
                for (int spin = 0; spin < a.spin_limit && missing; spin++) {
#pragma unroll
                    for (int v = 0; v < V; v++)
                        w[v] = __hip_atomic_load(slot + v * MAX_SEG + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    missing = false;
#pragma unroll
                    for (int v = 0; v < V; v++)
                        missing |= (uint32_t)(w[v] >> 32) != round;
                }
            if (theirs && !missing)
#pragma unroll
                for (int v = 0; v < V; v++)
                    s_part[at][v][lane] = __uint_as_float((uint32_t)w[v]);
            const bool any = __ballot(missing) != 0;
            if (lane == 0)
                s_missing[at] = any;
        } else {
            then();
        }
        __syncthreads();
        return s_missing[at] == 0;
    };
    auto part = [&](int v) __attribute__((always_inline)) { return lane < n_seg ? s_part[round & 1][v][lane] : 0.0f; };
    auto visit = [&](int n) __attribute__((always_inline)) {
        cur = n;
        depth++;
        if (wg == 0 && tid == 0)
            a.accept_path[(int64_t)b * (max_depth + 1) + depth] = cur;
        kids = __ballot(par_l == cur);
        have_mass = false;
    };

    bool known = true, in_time = true;                      // the current node's statistics are there; nobody was missing
    for (;;) {
        // ---- at a node whose children are all untried
        n_rej = 0;
        if (!kids) {
            // a leaf: (max, sum of exponentials) of its target row's segments
            round++;
            if (!messenger) {
                read_own(false);
                float m, z;
                wave_stats(rp, m, z);
                if (lane == 0) {
                    s_red[round & 1][0][wave] = m;
                    s_red[round & 1][1][wave] = z;
                }
            }
            in_time = exchange(std::integral_constant<int, 2>{}, [] {});
            mt = wave_max(lane < n_seg ? part(0) : -INFINITY);
            ip = 1.0f;
            const float zs = part(1);
            mass_l = zs > 0.0f ? zs * __expf(part(0) - mt) : 0.0f;
            have_mass = true;
            break;
        }
        if (!known) {
            // its rows' statistics, and the masses of its target's segments
            round++;
            if (!messenger) {
                read_own(true);
                float m, z, m2, z2;
                wave_stats(rp, m, z);
                wave_stats(rq, m2, z2);
                if (lane == 0) {
                    s_red[round & 1][0][wave] = m;
                    s_red[round & 1][1][wave] = z;
                    s_red[round & 1][2][wave] = m2;
                    s_red[round & 1][3][wave] = z2;
                }
            }
            in_time = exchange(std::integral_constant<int, 4>{}, [&] {
                if (depth < max_depth)
                    ask_rows(__builtin_ctzll(kids));
            });
            if (!in_time)
                break;
            const float m = lane < n_seg ? part(0) : -INFINITY, m2 = lane < n_seg ? part(2) : -INFINITY, z = part(1), z2 = part(3);
            mt = wave_max(m);                               // (lane s: segment s; the same tree over the segments in every wave)
            md = wave_max(m2);
            zt = wave_sum(z > 0.0f ? z * __expf(m - mt) : 0.0f);
            zd = wave_sum(z2 > 0.0f ? z2 * __expf(m2 - md) : 0.0f);
            mass_l = z > 0.0f ? z * __expf(m - mt) * (1.0f / zt) : 0.0f;
            have_mass = true;
        }
        ip = 1.0f / zt;
        iq = zd > 0.0f ? 1.0f / zd : 0.0f;
        if (depth >= max_depth)                             // (a node at the depth limit may have children)
            break;
        // ---- the first child against the untouched distributions
        const float px = __expf(tx_l - mt), qx = __expf(dx_l - md);
        const float ratio = qx > 0.0f ? (px / zt) / (qx / zd) : (px > 0.0f ? INFINITY : 0.0f);
        const uint64_t pass = __ballot(u_l < fminf(1.0f, ratio));
        int child = __builtin_ctzll(kids);
        kids &= kids - 1;
        bool accepted = pass >> child & 1;
        if (!accepted) {
            // ---- one rejection after the other: the target becomes the positive part of (target - draft), the token leaves the draft
            if (!messenger) {
                if (known)                                  // (otherwise the round before has read them)
                    read_own(true);
#pragma unroll
                for (int i = 0; i < PER * 8; i++) {
                    rp[i / 8][i % 8] = token_mass(rp[i / 8][i % 8], inv_temp, mt, ip);     // (0 past the end: the logits read as -inf there)
                    rq[i / 8][i % 8] = token_mass(rq[i / 8][i % 8], inv_temp, md, iq);
                }
            }
            float P_l = px * ip, Q_l = qx * iq, Zq = 1.0f, jp = 1.0f, jq = 1.0f, Zp = 1.0f;
            for (;;) {
                const int x = __builtin_amdgcn_readlane(tok_l, child), mine = x - t_own;
                round++;
                float r[PER][8];
                if (!messenger) {
                    float s = 0.0f;
#pragma unroll
                    for (int i = 0; i < PER * 8; i++) {
                        r[i / 8][i % 8] = residual(rp[i / 8][i % 8], jp, rq[i / 8][i % 8], jq);
                        s += r[i / 8][i % 8];
                    }
                    s = wave_sum(s);
                    if (lane == 0)
                        s_red[round & 1][0][wave] = s;
                }
                // what follows if something is left of the target
                const float rP_l = residual(P_l, jp, Q_l, jq);
                Zq = fmaxf(Zq - of_lane(Q_l, child), 0.0f);
                Q_l = tok_l == x ? 0.0f : Q_l;
                const int next = kids ? __builtin_ctzll(kids) : -1;
                const float Qn = of_lane(Q_l, next & 63), un = of_lane(u_l, next & 63), Pn = of_lane(rP_l, next & 63), qn = Qn / Zq;
                in_time = exchange(std::integral_constant<int, 1>{}, [&] {
                    if (tid == 0)
                        s_step[n_rej] = {jp, jq, x, 1};
#pragma unroll
                    for (int i = 0; i < PER * 8; i++)
                        rq[i / 8][i % 8] = mine == i / 8 * (NT * 8) + i % 8 ? 0.0f : rq[i / 8][i % 8];
                    // (rows on their way slow the polls down, so only if the test passes should half of the target be left)
                    if (next >= 0 && un * qn < 2.0f * Pn)
                        ask_rows(next);
                });
                if (!in_time)
                    break;
                left_l = part(0);
                const float Z = wave_sum(left_l);
                const bool take = Z > 0.0f;
                if (take) {
                    Zp = Z;
                    have_mass = true;
                    mass_l = left_l;
                    P_l = rP_l;
#pragma unroll
                    for (int i = 0; i < PER * 8; i++)
                        rp[i / 8][i % 8] = r[i / 8][i % 8];
                } else if (tid == 0) {
                    s_step[n_rej].take = 0;                 // target == draft: the residual is empty and the target stays as it is
                }
                n_rej++;
                child = next;
                if (child < 0)
                    break;
                kids &= kids - 1;
                jp = 1.0f / Zp;
                jq = Zq > 0.0f ? 1.0f / Zq : 0.0f;
                const float P = of_lane(P_l, child), again = Qn > 0.0f ? (P / Zp) / qn : (P > 0.0f ? INFINITY : 0.0f);
                accepted = un < fminf(1.0f, again);
                if (accepted)
                    break;
            }
        }
        if (!accepted)
            break;
        visit(child);
        known = !a.lazy;
        if (known) {
            mt = of_lane(mt_l, cur); zt = of_lane(zt_l, cur); md = of_lane(md_l, cur); zd = of_lane(zd_l, cur);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // (nothing is on its way to LDS when a wave ends)
    if (!in_time) {
        if (wg == 0 && !messenger)
            walk<BF16, PER, true, 64>(a);
        return;
    }
    // ---- no child, or every child rejected: draw from the current target
    if (wg != 0 || messenger)
        return;
    if (!have_mass) {                                       // the untouched target
        const float z = lane < n_seg ? a.stat_s[(bt + cur) * n_seg + lane] : 0.0f;
        mass_l = z > 0.0f ? z * __expf(a.stat_m[(bt + cur) * n_seg + lane] - mt) * ip : 0.0f;
    }
    // the segment with the drawn point is found from the masses, in order, and only that one is read
    float upto = mass_l;                                    // of the segments up to lane's
    for (int off = 1; off < 64; off <<= 1) {
        const float o = __shfl_up(upto, off);
        if (lane >= off)
            upto += o;
    }
    const float prev = __shfl_up(upto, 1), below_l = lane ? prev : 0.0f;
    const float target = u_bonus * of_lane(upto, 63);
    const uint64_t past = __ballot(mass_l > 0.0f && upto > target), some = __ballot(mass_l > 0.0f);
    // (rounding may leave the target at or above the total: the last segment with mass)
    const int pick = past ? __builtin_ctzll(past) : some ? 63 - __builtin_clzll(some) : 0;
    // Inverse-CDF draw over the segment's tokens, up to PER groups of 8 contiguous ones per thread: block scan, the thread with the drawn point goes over its own again.  Without one
    // (rounding left the target at or above the sum) the last token with mass is taken.
    const int r0 = pick * (PER * NT * 8), r1 = min(r0 + PER * NT * 8, vocab);
    const int cpt = ((r1 - r0 + NT - 1) / NT + 7) & ~7, t0 = min(r0 + tid * cpt, r1), t1 = min(t0 + cpt, r1);
    const int64_t row = (bt + cur) * vocab;
    Row rt[PER], rd[PER];
#pragma unroll
    for (int h = 0; h < PER; h++)
        if (t0 + h * 8 < t1) {
            rt[h].load(a.tlogits, row, t0 + h * 8, vocab);
            if (n_rej)
                rd[h].load(a.dlogits, row, t0 + h * 8, vocab);
        }
    float v[PER][8], local = 0.0f;
    __syncthreads();                                        // (the list of steps)
#pragma unroll
    for (int h = 0; h < PER; h++) {
#pragma unroll
        for (int j = 0; j < 8; j++)
            v[h][j] = 0.0f;
        if (t0 + h * 8 >= t1)
            continue;
        rt[h].unpack(v[h]);
#pragma unroll
        for (int j = 0; j < 8; j++)
            v[h][j] = token_mass(v[h][j], inv_temp, mt, ip);
        if (n_rej) {
            float dv[8];
            rd[h].unpack(dv);
#pragma unroll
            for (int j = 0; j < 8; j++)
                dv[j] = token_mass(dv[j], inv_temp, md, iq);
            Step s = s_step[0];
            for (int i = 0; i < n_rej; i++) {
                const Step after = s_step[min(i + 1, n_rej - 1)];
                const int x = s.x - t0 - h * 8;
                if (__builtin_amdgcn_readfirstlane(s.take))
#pragma unroll
                    for (int j = 0; j < 8; j++)
                        v[h][j] = residual(v[h][j], s.jp, dv[j], s.jq);
                if (__ballot((unsigned)x < 8))
#pragma unroll
                    for (int j = 0; j < 8; j++)
                        dv[j] = x == j ? 0.0f : dv[j];
                s = after;
            }
        }
#pragma unroll
        for (int j = 0; j < 8; j++)
            local += v[h][j];
    }
    float inc = local;   // inclusive scan of the per-thread sums: inside a wave by shuffles, wave totals through LDS
    for (int off = 1; off < 64; off <<= 1) {
        const float o = __shfl_up(inc, off);
        if (lane >= off)
            inc += o;
    }
    if (lane == 63)
        s_scan[wave] = inc;
    __syncthreads();
    float base = of_lane(below_l, pick);
#pragma unroll
    for (int w = 0; w < NW; w++)
        if (w < wave)
            base += s_scan[w];
    const float below = base + inc - local;                 // mass of all tokens below t0
    const uint64_t hit = __ballot(below + local > target && t1 > t0);
    int last = -1;                                          // the thread's last token with mass, then the wave's
#pragma unroll
    for (int i = 0; i < PER * 8; i++)
        last = v[i / 8][i % 8] > 0.0f ? t0 + i : last;
    const uint64_t any = __ballot(last >= 0);
    last = any ? __builtin_amdgcn_readlane(last, 63 - __builtin_clzll(any | 1)) : -1;
    if (lane == 0) {
        s_redi[wave] = hit ? wave * 64 + __builtin_ctzll(hit) : 0x7fffffff;
        s_last[wave] = last;
    }
    __syncthreads();
    int owner = 0x7fffffff;
    last = -1;
#pragma unroll
    for (int w = 0; w < NW; w++) {
        owner = min(owner, s_redi[w]);
        last = max(last, s_last[w]);
    }
    if (tid == owner) {
        float run = below;
        int token = t1 - 1;
        bool found = false;
#pragma unroll
        for (int i = 0; i < PER * 8; i++) {
            run += v[i / 8][i % 8];
            if (!found && run > target && t0 + i < t1) {
                token = t0 + i;
                found = true;
            }
        }
        a.bonus_token[b] = token;
    }
    if (tid == 0) {
        if (owner == 0x7fffffff)
            a.bonus_token[b] = last >= 0 ? last : min(r0, vocab - 1);
        a.accept_len[b] = depth;
    }
}

}  // namespace

extern "C" {

size_t dream_spec_accept_workspace(int32_t batch, int32_t n_tree, int32_t vocab)
{
    if (batch < 1 || n_tree < 1 || vocab < 1)
        return DREAM_WORKSPACE_MIN_BYTES;
    // The size is part of the boundary: programs hold it as a number.  Of it the calls use the statistics' two arrays and SLOTS words per
    // sequence, which sit where an earlier form of the walk kept three vocabulary rows; the rest is not touched.
    const size_t stats = align_up((size_t)2 * batch * n_tree * ceil_div(vocab, 8192) * sizeof(float), 256);
    return DREAM_WORKSPACE_MIN_BYTES + align_up((size_t)batch * 3 * vocab * sizeof(float), 256) + 3 * stats + align_up((size_t)batch * n_tree * 4 * sizeof(float), 256);
}

int dream_spec_accept(const void *target_logits, const void *draft_logits, int32_t logits_dtype, int32_t batch, int32_t n_tree,
                      int32_t vocab, const int32_t *token, const int32_t *parent, const float *u_accept, const float *u_bonus,
                      int32_t max_depth, float temperature, int32_t *accept_len, int32_t *accept_path, int32_t *bonus_token,
                      void *workspace, size_t workspace_bytes, void *stream)
{
    const char *who = "dream_spec_accept";
    if (!target_logits || !draft_logits || !token || !parent || !u_accept || !u_bonus || !accept_len || !accept_path || !bonus_token)
        return fail(DREAM_ERR_INVALID_ARG, "%s: NULL argument", who);
    if (logits_dtype != DREAM_F32 && logits_dtype != DREAM_BF16)
        return fail(DREAM_ERR_INVALID_ARG, "%s: unknown logits dtype %d", who, logits_dtype);
    if (batch < 1 || batch > 65535 || vocab < 1 || max_depth < 0 || max_depth >= DREAM_MAX_TREE_ACCEPT)
        return fail(DREAM_ERR_INVALID_ARG, "%s: batch in [1, 65535], vocab positive and 0 <= max_depth < %d required", who, DREAM_MAX_TREE_ACCEPT);
    if (n_tree < 1 || n_tree > DREAM_MAX_TREE_ACCEPT)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: n_tree %d outside [1, %d]", who, n_tree, DREAM_MAX_TREE_ACCEPT);
    if ((int64_t)batch * n_tree > 65535)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: batch * n_tree = %lld exceeds 65535 rows", who, (long long)batch * n_tree);
    if (!(temperature > 0.0f))
        return fail(DREAM_ERR_INVALID_ARG, "%s: temperature must be positive (use dream_accept_path for the greedy rule)", who);
    const size_t need = dream_spec_accept_workspace(batch, n_tree, vocab);
    if (!workspace || workspace_bytes < need)
        return fail(DREAM_ERR_WORKSPACE, "%s: workspace of %zu bytes, %zu needed", who, workspace_bytes, need);
    int per = 1;
    while (per < 4 && ceil_div(vocab, NT * 8 * per) > std::min(MAX_SEG, std::max(1, 256 / batch)))
        per *= 2;
    const int n_chunks = ceil_div(vocab, NT * 8 * per);
    const size_t stats = align_up((size_t)2 * batch * n_tree * n_chunks * sizeof(float), 256);
    // Workgroups per sequence: one per segment while all of them together stay within one per CU.
    const int seg_chunks = ceil_div(n_chunks, MAX_SEG), n_seg = ceil_div(n_chunks, seg_chunks);
    const int n_wg = std::max(1, std::min(n_seg, 256 / batch));
    // the slots exist with more than one segment only, so they fit where a row of floats per sequence does, and the statistics in the other two
    // (aligned here, in the room the first DREAM_WORKSPACE_MIN_BYTES leave: a slot is one 64-bit word to readers and writers only where it is aligned)
    char *wsb = reinterpret_cast<char *>(align_up(reinterpret_cast<uintptr_t>(workspace), DREAM_WORKSPACE_MIN_BYTES));
    uint64_t *slots = n_wg > 1 ? reinterpret_cast<uint64_t *>(wsb) : nullptr;
    const size_t slot_bytes = n_wg > 1 ? (size_t)batch * SLOTS * sizeof(uint64_t) : 0;
    float *stat_m = reinterpret_cast<float *>(wsb + slot_bytes);
    float *stat_s = reinterpret_cast<float *>(wsb + slot_bytes + stats);
    if (align_up(reinterpret_cast<uintptr_t>(workspace), DREAM_WORKSPACE_MIN_BYTES) - reinterpret_cast<uintptr_t>(workspace) + slot_bytes + 2 * stats > need)
        return fail(DREAM_ERR_WORKSPACE, "%s: the statistics do not fit the workspace", who);
    const int esz = logits_dtype == DREAM_BF16 ? 2 : 4;
    const bool vec = vocab % 8 == 0 &&
                     ((reinterpret_cast<uintptr_t>(target_logits) | reinterpret_cast<uintptr_t>(draft_logits)) & 15) == 0 &&
                     ((size_t)vocab * esz) % 16 == 0;
    const float inv_temp = 1.0f / temperature;
    hipStream_t st = as_stream(stream);
    // The statistics of all nodes beforehand cost a read of about half of all rows, those of the visited ones an exchange each, which also brings the rows
    // that the rejections there need.  A small tree has as many levels to visit for its bytes as a large one and fewer rejections on the way, so
    // the line is one of bytes times nodes, with a floor for large trees.  us, all / visited, the same tensors every call; then several sets in turn, 1 GB and
    // more: 8 nodes, 134 MB of logits 37 / 50; 42 / 55, 268 MB 60 / 65; 67 / 70; 16 nodes, 134 MB 35 / 43; 38 / 44, 201 MB 48 / 48; 55 / 49, 268 MB
    // 52 / 46; 59 / 50; 24 nodes, 101 MB 33 / 41; 37 / 43, 151 MB 39 / 39; 42 / 41, 201 MB 43 / 43; 47 / 46; 32 nodes, 67 MB 33 / 36; 35 / 37, 134 MB 43 / 42;
    // 45 / 43; 48 nodes, 50 MB 27 / 37; 29 / 34, 75 MB 36 / 36; 39 / 39, 101 MB 38 / 38; 43 / 39; 64 nodes, 50 MB 42 / 44; 37 / 41, 67 MB 29 / 29; 31 / 31,
    // 134 MB 48 / 44; 53 / 48.  Over 262 shapes of 40 to 500 MB, 8 to 64 nodes and 1 to 32 sequences the line takes 0.5 % more than the better of both on average, 16 % at
    // worst (bytes alone, 60 MB: 4.7 %, 53 %).  spec_walk_small_kernel visits nodes for less and changes at 1.2 GB of bytes times nodes: 8 nodes, 67 MB 21 / 28, 134 MB 31 / 31 to 33;
    // 12 nodes, 50 MB 22 / 24, 101 MB 26 / 26; 16 nodes, 34 MB 19 / 19 and 20 / 24, 67 MB 24 / 21, 134 MB 29 / 25; 24 nodes, 25 MB 19 / 20, 50 MB 23 / 22 and 24 / 26, 101 MB 27 / 23;
    // 33 nodes, 17 MB 19 / 23, 35 MB 26 / 20 and 29 / 28, 138 MB 31 / 25; 60 nodes, 8 MB 23 / 25, 31 MB 34 / 29, 252 MB 50 / 30, 503 MB 71 / 30.
    const int64_t logit_bytes = (int64_t)2 * batch * n_tree * vocab * esz;
    const bool small = per <= 2 && n_tree <= 64 && n_chunks <= n_wg;        // (with four groups a thread the registers do not suffice for a ninth wave)
    const bool lazy = small ? logit_bytes * n_tree >= 1200000000ll : logit_bytes >= 60000000 && logit_bytes * n_tree >= 3000000000ll;
    const int n_nodes = lazy ? 1 : n_tree;
    const dim3 sgrid(n_chunks, batch * n_nodes, 2);
    const WalkArgs wa = {target_logits, draft_logits, n_tree, vocab, n_chunks, seg_chunks, n_seg, vec ? 1 : 0, lazy ? 1 : 0, token, parent, u_accept, u_bonus, max_depth,
                         inv_temp, accept_spin_limit(), stat_m, stat_s, slots, accept_len, accept_path, bonus_token};
    auto launch_all = [&](auto bf16, auto groups) {
        constexpr bool BF = decltype(bf16)::value;
        constexpr int PER = decltype(groups)::value;
        hipLaunchKernelGGL((softmax_stats_kernel<BF, PER>), sgrid, dim3(256), 0, st, target_logits, draft_logits, n_tree, n_nodes, vocab, n_chunks, vec ? 1 : 0,
                           parent, inv_temp, stat_m, stat_s, slots, (int64_t)batch * n_tree);
        if constexpr (PER <= 2) {
            if (small) {
                if (vec)
                    hipLaunchKernelGGL((spec_walk_small_kernel<BF, PER, true>), dim3(n_wg, batch), dim3(NT + 64), 0, st, parent, token, u_accept, u_bonus, target_logits, draft_logits, n_tree, vocab, wa);
                else
                    hipLaunchKernelGGL((spec_walk_small_kernel<BF, PER, false>), dim3(n_wg, batch), dim3(NT + 64), 0, st, parent, token, u_accept, u_bonus, target_logits, draft_logits, n_tree, vocab, wa);
                return;
            }
        }
        hipLaunchKernelGGL((spec_walk_kernel<BF, PER>), dim3(n_wg, batch), dim3(NT), 0, st, wa);
    };
    auto with_groups = [&](auto bf16) {
        if (per == 1)
            launch_all(bf16, std::integral_constant<int, 1>{});
        else if (per == 2)
            launch_all(bf16, std::integral_constant<int, 2>{});
        else
            launch_all(bf16, std::integral_constant<int, 4>{});
    };
    if (logits_dtype == DREAM_BF16)
        with_groups(std::true_type{});
    else
        with_groups(std::false_type{});
    return check_launch("spec_accept kernels");
}

}  // extern "C"
