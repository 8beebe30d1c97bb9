// Tree-masked attention kernels for gfx950: dream_tree_verify_attn and dream_draft_xattn.
//
// Both calls compute softmax(q k^T * scale) v (Section 3.1, Eq. 1) over the keys a tree node may
// see: the whole cached prefix plus its ancestors in the draft tree (Section 3.1, tree-masking
// paragraph); verification includes the node itself, the draft's cross-attention does not.
//
// bf16, shared tiles (attn_bf16_kernel).  A workgroup serves one (sequence, KV head, key-range split, query
// group).  The query rows that share a KV head - every tree row of every query head of the GQA
// group - are cut into 16-row tiles; each wave owns QG of them (4 waves, or 8 waves for grouped-query shapes, or
// 8 waves as two key groups where a CU gets one workgroup).  All threads stream the key range in
// 32-key K/V tiles with 16-byte coalesced loads kept one or two steps ahead in registers, park each tile in one of
// two LDS stages (one barrier per step), and every wave reads the tile's MFMA fragments from LDS: a K/V byte leaves
// HBM once and serves all tree rows and all heads of the group.  Scores are formed transposed, S^T = K Q^T, with
// v_mfma_f32_16x16x32_bf16, so a lane owns one query column: the online-softmax state is a
// per-lane scalar and the fp32 score registers, converted to bf16, already are the B operand of
// the second contraction O^T += V^T P^T, whose A operand (V transposed) comes from the LDS
// transpose read ds_read_b64_tr_b16.  The softmax reference of a column is raised only when a
// score exceeds it by 8 octaves, so accumulators are rescaled a handful of times per call.  Where a workgroup is the
// only reader of its K/V rows the loads carry the nontemporal hint; output rows leave as whole lines with it.
//
// bf16, few streams (attn_wave_kernel, attn_pair_kernel, attn_quad_kernel).  A CU pulls at most about 65 GB/s through its L1, so a short stream is
// bandwidth-starved unless all 256 CUs pull a share of it.  While at most one workgroup per CU comes of it, the work of a KV head is cut into
// query tiles and column slices only: a workgroup's waves stream disjoint key tiles, straight to LDS, and their states meet in LDS at
// the end, in one launch.  Beyond the lengths where that pays, the key range is split over several workgroups of attn_bf16_kernel, each
// writes its (reference, sum, O) state to the workspace, and attn_merge_kernel merges the states of a group in split order
// (deterministic) and writes the rows.  (A merge across workgroups inside one launch costs more than the second launch: the L2s of
// the XCDs are not coherent with each other.)  Workgroups that read the same K/V stream get ids congruent mod 8 so that they run on
// one XCD and share its L2.
//
// fp32 path (attn_f32_kernel): vector-ALU kernel, one workgroup per (query row, head, sequence), used for float32
// tensors (the small configuration).
#include "common.h"
#include "dream_tuning.h"
#include "lds_tiles.h"
#include <math.h>
#include <type_traits>

using namespace dream;

namespace {

struct AttnArgs {
    const void *q, *k, *v;
    const int32_t *prefix_len, *parent, *q_node;
    const uint64_t *tree_mask;   // [B, n_tree, mask_words] when given
    void *out;
    float *lse;
    float *part;             // [groups, splits, 4 waves, state] per-wave states of every split
    int32_t n_q_heads, n_kv_heads, group;
    int32_t n_q;
    uint32_t spread;         // attend_rows: ceil(2^16 / Hkv) where the KV heads of all sequences are numbered together, 0 where Hkv is a multiple of 8
    int32_t n_tree, include_self;
    union {
        int32_t tiles_per_head;  // 16-row query tiles per head (attn_bf16_kernel)
        uint32_t turn;           // attend_rows: 2^16 * TURN / workgroups of a KV head where the order of RowsGeom::TURNED or SWAPPED is used, or 0
    };
    int32_t n_qg;            // query groups per KV head
    int32_t mask_words;      // 64-bit words of a node's visibility mask: ceil(n_tree / 64)
    int32_t n_splits;
    int32_t n_streams;       // B * Hkv * n_splits
    int64_t s_max;
    float scale, scale_log2;
    uint32_t nq_magic;       // for quick_div by n_q
    int32_t once;            // the caches will not be read again before others have displaced them (the ONCE forms of attend_rows)
};

// Visibility of the tree nodes to one query: bit (a % 64) of word a / 64 is set iff node a is visible.  MW = 1 serves
// trees of up to 64 nodes, MW = 4 up to 256.
template <int MW>
struct NodeMask {
    uint64_t w[MW];
};

template <int MW>
__device__ __forceinline__ void mask_set(NodeMask<MW> &m, int node)
{
    if (MW == 1) {
        m.w[0] |= 1ull << node;
    } else {
#pragma unroll
        for (int i = 0; i < MW; i++)
            m.w[i] |= (node >> 6) == i ? 1ull << (node & 63) : 0ull;
    }
}

// bit `rel` of the mask (the caller has already excluded rel outside [0, n_tree))
template <int MW>
__device__ __forceinline__ uint32_t mask_bit(const NodeMask<MW> &m, int rel)
{
    if (MW == 1)
        return (uint32_t)(m.w[0] >> (rel & 63)) & 1u;
    // (kept as arithmetic on all words: a per-lane choice of the word would become an indexed private array)
    uint32_t bit = 0u;
#pragma unroll
    for (int i = 0; i < MW; i++)
        bit |= (uint32_t)(m.w[i] >> (rel & 63)) & (uint32_t)((rel >> 6) == i);
    return bit & 1u;
}

template <int MW>
__device__ __forceinline__ NodeMask<MW> visible_nodes(const AttnArgs &a, int b, int node, const int32_t *lds_parent)
{
    NodeMask<MW> m;
#pragma unroll
    for (int i = 0; i < MW; i++)
        m.w[i] = 0ull;
    if (a.tree_mask) {
#pragma unroll
        for (int i = 0; i < MW; i++)
            if (i < a.mask_words)
                m.w[i] = a.tree_mask[((int64_t)b * a.n_tree + node) * a.mask_words + i];
        return m;
    }
    if (a.include_self)
        mask_set(m, node);
    for (int p = lds_parent[node]; p >= 0; p = lds_parent[p])
        mask_set(m, p);
    return m;
}

template <int MW>
__device__ __forceinline__ NodeMask<MW> empty_mask()
{
    NodeMask<MW> m;
#pragma unroll
    for (int i = 0; i < MW; i++)
        m.w[i] = 0ull;
    return m;
}

template <int D, int QG, int KT>
struct Geom {
    static constexpr int KSTR = D + 8;    // K row stride in LDS (elements): 16-byte pad, b128 reads spread over all banks
    static constexpr int VSTR = D + 16;  // V row stride in LDS (elements): 4 consecutive rows land 8 banks apart
    static constexpr int TILE_ELEMS = 32 * (KSTR + VSTR);   // one 32-key K tile followed by its V tile
    static constexpr int STAGE_ELEMS = KT * TILE_ELEMS;     // a step handles KT tiles
    static constexpr int NDT = D / 16;
    static constexpr int NKS = D / 32;
    static constexpr int CH = 32 * D / 8 / 256;             // 16-byte chunks per thread per tensor per tile
    static constexpr size_t LDS_BYTES = (size_t)2 * STAGE_ELEMS * 2 + DREAM_MAX_TREE * sizeof(int32_t);
};

template <int D, int QG>
struct StateGeom {
    static constexpr int NDT = D / 16;
    static constexpr int STATE_FLOATS = QG * NDT * 256 + QG * 2 * 64;   // one wave's (O, reference, sum) in lane-major order
};

template <int QG, int NDT>
struct WaveState {
    f32x4 o[QG][NDT];
    float m[QG], l[QG];
};

template <int QG, int NDT>
__device__ __forceinline__ void state_store(const WaveState<QG, NDT> &s, float *dst, int lane)
{
#pragma unroll
    for (int qt = 0; qt < QG; qt++) {
#pragma unroll
        for (int dt = 0; dt < NDT; dt++)
            reinterpret_cast<f32x4 *>(dst)[(qt * NDT + dt) * 64 + lane] = s.o[qt][dt];
        dst[QG * NDT * 256 + (qt * 2) * 64 + lane] = s.m[qt];
        dst[QG * NDT * 256 + (qt * 2 + 1) * 64 + lane] = s.l[qt];
    }
}

// Row ownership of a lane: query tile qt of wave `wave` in query group qg -> (query head, query row) of column c.
struct RowOwner {
    int row, head;
};
__device__ __forceinline__ RowOwner row_owner(const AttnArgs &a, int kvh, int qg, int wave, int QG, int qt, int c, int nw = 4)
{
    int tq = (qg * nw + wave) * QG + qt;
    int hh = tq / a.tiles_per_head, nt = tq % a.tiles_per_head;
    int row = nt * 16 + c;
    bool valid = tq < a.group * a.tiles_per_head && row < a.n_q;
    RowOwner r;
    r.row = valid ? row : -1;
    r.head = kvh * a.group + hh;
    return r;
}

// The softmax reference of a column is only raised when a score exceeds it by more than this many
// octaves, so exp2(score - reference) stays below 2^8 and the accumulators are seldom rescaled.
#define DREAM_SOFTMAX_SLACK 8.0f
// Build-time knobs of the launch shapes (each value is the measured best):
#ifndef DREAM_Q1_WAVES
#define DREAM_Q1_WAVES 2     // waves per SIMD the 4-wave one-tile-per-wave variants are compiled for (3: 1024 workgroups then run as 3 + 1 per CU, 75 against 71 us at 32 LLaVA sequences; 4: spills)
#endif
#ifndef DREAM_KG2_MAX_WG
#define DREAM_KG2_MAX_WG 1   // two key groups while a CU would get at most this many 4-wave workgroups (measured: -5 % at 1, +3 % at 4)
#endif
#ifndef DREAM_W8Q1_WAVES
#define DREAM_W8Q1_WAVES 1   // the same for the 8-wave variants (2 workgroups per CU would need 128 registers: spills, slower)
#endif
#ifndef DREAM_W8_PFD
#define DREAM_W8_PFD 2   // steps in flight of the 8-wave shared-tile form
#endif


// Online softmax of KT 32-key tiles for the QG query tiles of a wave.  sacc holds the raw scores S^T (lane owns
// query column c and key rows g*4+r of every 16-key block); on return pf holds the probabilities as the bf16 B
// operand of O^T += V^T P^T, and the running (reference, sum, accumulators) of `st` are updated.
// Only the first part depends on whether the step needs the visibility test (one wave-uniform branch per step, not
// one per score): a step wholly inside the prefix takes the maximum over the raw scores and leaves the scaling to
// the exponent's fused multiply-add; the general path scales and masks the scores in place.
// softmax_prepare: visibility test, maxima, and the (rare) raise of the references with the rescaling of the
// accumulators; returns what still multiplies the stored scores.  softmax_exponentials: the straight-line rest.
template <int QG, int KT, int NDT, int MW>
__device__ __forceinline__ float softmax_prepare(f32x4 (&sacc)[KT][2][QG], WaveState<QG, NDT> &st, const NodeMask<MW> (&qmask)[QG],
                                                 bool needs_mask, int key0, int P, int key_end, int n_tree, float scale_log2, int g)
{
    float mx_q[QG];
    if (needs_mask) {
#pragma unroll
        for (int qt = 0; qt < QG; qt++) {
            float mx = -INFINITY;
#pragma unroll
            for (int kt = 0; kt < KT; kt++) {
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    float x = sacc[kt][e >> 2][qt][e & 3] * scale_log2;
                    const int key = key0 + kt * 32 + (e >> 2) * 16 + g * 4 + (e & 3);
                    const int rel = key - P;
                    const uint32_t bit = mask_bit(qmask[qt], rel);
                    const uint32_t vis = ((uint32_t)(rel < 0) | ((uint32_t)(rel < n_tree) & bit)) & (uint32_t)(key < key_end);
                    x = vis ? x : -INFINITY;
                    sacc[kt][e >> 2][qt][e & 3] = x;
                    mx = fmaxf(mx, x);
                }
            }
            mx_q[qt] = mx;
        }
    } else {
#pragma unroll
        for (int qt = 0; qt < QG; qt++) {
            float mx = -INFINITY;
#pragma unroll
            for (int kt = 0; kt < KT; kt++)
#pragma unroll
                for (int e = 0; e < 8; e++)
                    mx = fmaxf(mx, sacc[kt][e >> 2][qt][e & 3]);
            mx_q[qt] = mx * scale_log2;   // scale_log2 >= 0 on this path
        }
    }
    const float mult = needs_mask ? 1.0f : scale_log2;   // what still multiplies the stored scores
    bool raise = false;
#pragma unroll
    for (int qt = 0; qt < QG; qt++)
        raise = raise || (mx_q[qt] > st.m[qt] + DREAM_SOFTMAX_SLACK);
    if (__any(raise)) {
        // rare: some column's reference is raised to the true maximum over its 4 row groups
#pragma unroll
        for (int qt = 0; qt < QG; qt++) {
            float mx = mx_q[qt];
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            if (mx > st.m[qt] + DREAM_SOFTMAX_SLACK) {
                float alpha = __builtin_amdgcn_exp2f(st.m[qt] - mx);   // 0 when the old reference was -inf
                st.m[qt] = mx;
                st.l[qt] *= alpha;
#pragma unroll
                for (int dt = 0; dt < NDT; dt++)
                    st.o[qt][dt] *= alpha;
            }
        }
    }
    return mult;
}

template <int QG, int KT, int NDT>
__device__ __forceinline__ void softmax_exponentials(const f32x4 (&sacc)[KT][2][QG], bf16x8 (&pf)[KT][QG], WaveState<QG, NDT> &st, float mult)
{
#pragma unroll
    for (int qt = 0; qt < QG; qt++) {
        const float neg_m = (st.m[qt] == -INFINITY) ? 0.0f : -st.m[qt];
        float psum = 0.0f;
#pragma unroll
        for (int kt = 0; kt < KT; kt++) {
#pragma unroll
            for (int e = 0; e < 8; e++) {
                float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kt][e >> 2][qt][e & 3], mult, neg_m));
                psum += p;
                pf[kt][qt][e] = (__bf16)p;
            }
        }
        st.l[qt] += psum;
    }
}

// S^T = K Q^T for the KT 32-key tiles held in LDS at `stage` (K tile, then V tile, per 32 keys) x the (16 * QG) query
// columns of this wave; independent accumulators keep the MFMA pipe full.
template <int D, int QG, int KT>
__device__ __forceinline__ void tiles_scores(const uint16_t *stage, const bf16x8 (&qf)[QG][D / 32], f32x4 (&sacc)[KT][2][QG], int c, int g)
{
    using G = Geom<D, QG, KT>;
    constexpr int KSTR = G::KSTR, NKS = G::NKS;
#pragma unroll
    for (int kt = 0; kt < KT; kt++) {
        const uint16_t *sk = stage + kt * G::TILE_ELEMS;
        bf16x8 kfr[2][NKS];
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
            kfr[0][ks] = *reinterpret_cast<const bf16x8 *>(sk + c * KSTR + ks * 32 + g * 8);
            kfr[1][ks] = *reinterpret_cast<const bf16x8 *>(sk + (16 + c) * KSTR + ks * 32 + g * 8);
        }
#pragma unroll
        for (int qt = 0; qt < QG; qt++) {
            sacc[kt][0][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
            sacc[kt][1][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int ks = 0; ks < NKS; ks++) {
#pragma unroll
            for (int qt = 0; qt < QG; qt++) {
                sacc[kt][0][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kfr[0][ks], qf[qt][ks], sacc[kt][0][qt], 0, 0, 0);
                sacc[kt][1][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kfr[1][ks], qf[qt][ks], sacc[kt][1][qt], 0, 0, 0);
            }
        }
    }
}

// Online softmax of the raw scores `sacc` of the KT tiles at `stage` (first key key0) and O^T += V^T P^T.
template <int D, int QG, int KT, int MW>
__device__ __forceinline__ void tiles_softmax_pv(const uint16_t *stage, int key0, int P, int key_end, int n_tree, float scale_log2,
                                                 f32x4 (&sacc)[KT][2][QG], const NodeMask<MW> (&qmask)[QG], WaveState<QG, D / 16> &st, int c, int g)
{
    using G = Geom<D, QG, KT>;
    constexpr int KSTR = G::KSTR, VSTR = G::VSTR, NDT = G::NDT;
    // step touches tree rows, the ragged end or the next split (a negative scale also goes the general way)
    const bool needs_mask = key0 + KT * 32 > min(P, key_end) || scale_log2 < 0.0f;
    // ---- V^T fragments of the first tile (first half of the head dimension for D = 256) are requested
    // now, so their LDS latency hides behind the softmax arithmetic
    constexpr int VH = D == 256 ? 2 : 1, NDH = NDT / VH;
    s16x4 vfr[NDH][2];
    const int v_off = 32 * KSTR + (g * 4 + (c >> 2)) * VSTR + (c & 3) * 4;
    auto read_v = [&](int kt, int h) {
        const uint16_t *vrow = stage + kt * G::TILE_ELEMS + v_off + h * NDH * 16;
#pragma unroll
        for (int dt = 0; dt < NDH; dt++) {
            vfr[dt][0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(vrow + dt * 16));
            vfr[dt][1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(vrow + dt * 16 + 16 * VSTR));
        }
    };
    read_v(0, 0);
    // ---- online softmax; lane owns query column c and key rows g*4+r of every 16-key block
    bf16x8 pf[KT][QG];
    const float mult = softmax_prepare<QG, KT, NDT, MW>(sacc, st, qmask, needs_mask, key0, P, key_end, n_tree, scale_log2, g);
    softmax_exponentials<QG, KT, NDT>(sacc, pf, st, mult);
    // ---- O^T += V^T P^T
#pragma unroll
    for (int kt = 0; kt < KT; kt++) {
#pragma unroll
        for (int h = 0; h < VH; h++) {
            if (kt > 0 || h > 0)
                read_v(kt, h);
#pragma unroll
            for (int dt = 0; dt < NDH; dt++) {
                s16x8 vv = __builtin_shufflevector(vfr[dt][0], vfr[dt][1], 0, 1, 2, 3, 4, 5, 6, 7);
                bf16x8 vf = __builtin_bit_cast(bf16x8, vv);
#pragma unroll
                for (int qt = 0; qt < QG; qt++)
                    st.o[qt][h * NDH + dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[kt][qt], st.o[qt][h * NDH + dt], 0, 0, 0);
            }
        }
    }
}

// QK^T, online softmax and PV for KT consecutive 32-key tiles held in LDS at `stage`, for the QG query tiles of this
// wave.  key0 is the global key index of the first row.
template <int D, int QG, int KT, int MW>
__device__ __forceinline__ void tiles_compute(const uint16_t *stage, int key0, int P, int key_end, int n_tree, float scale_log2,
                                              const bf16x8 (&qf)[QG][D / 32], const NodeMask<MW> (&qmask)[QG],
                                              WaveState<QG, D / 16> &st, int c, int g)
{
    f32x4 sacc[KT][2][QG];
    tiles_scores<D, QG, KT>(stage, qf, sacc, c, g);
    __builtin_amdgcn_sched_barrier(0);
    tiles_softmax_pv<D, QG, KT, MW>(stage, key0, P, key_end, n_tree, scale_log2, sacc, qmask, st, c, g);
}

// KT: 32-key tiles handled per step (per barrier, per softmax update); PFD: steps kept in flight in registers;
// NW: waves per workgroup (4, or 8 when the key range is not split: twice the query tiles share one LDS tile);
// MW: 64-bit words of a node's visibility mask (1: trees of up to 64 nodes; 4: up to 256);
// ONCE: this workgroup is the only reader of its K/V rows (one query group per KV head), so the loads carry the
// nontemporal hint: rows that are used once otherwise displace each other, and the output rows on their way out, in
// L2 (measured at 32 sequences: LLaVA 82.5 -> 71 us, SmolVLM 83.5 -> 74.5 us per launch).  With several query groups per
// KV head the later groups hit the rows in L2, so those launches use the variant without the hint.  (A run-time choice
// between the two kinds of load does not survive the compiler: it merges them into plain loads.)
template <int QG, int NDT>
__device__ __forceinline__ void state_merge(WaveState<QG, NDT> &s, const float *src, int lane);

// KG: key groups (1 or 2).  With 2, the 8 waves are two groups of 4: both serve the same (up to 4·QG) query tiles, a step
// stages 2·KT tiles and each group computes its KT of them; the two partial states of a query tile meet in LDS at the
// end.  Where a CU gets at most one workgroup: twice the waves and twice the bytes in flight.
template <int D, int QG, int KT, int PFD, int NW = 4, int MW = 1, bool ONCE = false, int KG = 1>
__global__ __launch_bounds__(64 * NW, (QG == 1 && D <= 128) ? (NW == 4 ? DREAM_Q1_WAVES : DREAM_W8Q1_WAVES) : 1) void attn_bf16_kernel(AttnArgs a)
{
    using G = Geom<D, QG, KT>;
    using GS = Geom<D, QG, KT * KG>;             // what a step stages
    static_assert(KG == 1 || (KG == 2 && NW == 8), "two key groups: 8 waves");
    constexpr int KSTR = G::KSTR, VSTR = G::VSTR, NDT = G::NDT, NKS = G::NKS;
    constexpr int QW = NW / KG;                  // waves that own different query tiles
    constexpr int NT = 64 * NW, LPR = D / 8, CPT = 32 * LPR;   // threads; 16-byte chunks per row and per tile (one tensor)
    constexpr int NLD = KT * KG * CPT / NT;                    // chunks per thread per tensor per step
    static_assert(NLD >= 1 && NLD * NT == KT * KG * CPT, "the chunks of a step divide evenly among the threads");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    uint16_t *lds = reinterpret_cast<uint16_t *>(smem_raw);
    int32_t *lds_parent = reinterpret_cast<int32_t *>(smem_raw + (size_t)2 * GS::STAGE_ELEMS * 2);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps bookkeeping in scalar registers
    const int wave = wave_all % QW, kgrp = wave_all / QW;             // query-tile slot and key group of this wave
    const int c = lane & 15, g = lane >> 4;

    // workgroup id -> (K/V stream, query group): ids that share a stream are congruent mod 8 (same XCD)
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int stream = (slot / a.n_qg) * 8 + xcd, qg = slot % a.n_qg;
    if (stream >= a.n_streams)
        return;
    const int nsplit = a.n_splits;
    const int split = stream % nsplit, bk = stream / nsplit;
    const int kvh = bk % a.n_kv_heads, b = bk / a.n_kv_heads;

    // tree metadata is requested first: the mask walk then overlaps the K/V loads still in flight
    int32_t my_parent = -1;
    if (!a.tree_mask && tid < a.n_tree)
        my_parent = a.parent[(int64_t)b * a.n_tree + tid];

    const int P = (int)min((int64_t)max(a.prefix_len[b], 0), a.s_max - a.n_tree);   // never past the cache, whatever the array holds
    const int kv_len = P + a.n_tree;
    const int tiles_total = (kv_len + 31) / 32;
    const int tps = (tiles_total + nsplit - 1) / nsplit;
    const int t_begin = split * tps;
    const int t_end = min(t_begin + tps, tiles_total);
    const int n_my = max(t_end - t_begin, 0);
    const int n_steps = (n_my + KT * KG - 1) / (KT * KG);
    const int key_end = min(kv_len, t_end * 32);   // keys at or past it belong to nobody or to the next split

    const uint16_t *kbase = reinterpret_cast<const uint16_t *>(a.k) + ((int64_t)b * a.n_kv_heads + kvh) * a.s_max * D;
    const uint16_t *vbase = reinterpret_cast<const uint16_t *>(a.v) + ((int64_t)b * a.n_kv_heads + kvh) * a.s_max * D;

    // ---- cooperative loads: a thread owns NLD 16-byte chunks of K and of V per step.  Rows past the live
    // range are clamped to the last live row (their scores are masked, so only finite values ever meet a
    // zero probability); tile indices past this workgroup's range are clamped too, so the number of loads
    // issued never depends on control flow and prefetches stay in flight across iterations.
    u32x4 kreg[PFD][NLD], vreg[PFD][NLD];
    // chunk j of this thread within a step: tile ld_tile(j) of the step, row ld_row(j), 16-byte column ld_col(j)
    // (a tile is CPT / NT passes of the workgroup, or, with more threads than a tile has chunks, a pass covers NT / CPT tiles)
    auto ld_tile = [&](int j) {
        if constexpr (CPT >= NT)
            return j / (CPT / NT);
        else
            return tid / CPT + j * (NT / CPT);
    };
    auto ld_row = [&](int j) {
        if constexpr (CPT >= NT)
            return tid / LPR + (j % (CPT / NT)) * (NT / LPR);
        else
            return (tid % CPT) / LPR;
    };
    const int ld_col = tid % LPR;   // (NT is a multiple of LPR)
    auto load_step = [&](int i, u32x4(&kr)[NLD], u32x4(&vr)[NLD]) {
#pragma unroll
        for (int j = 0; j < NLD; j++) {
            const int t = min(t_begin + i * KT * KG + ld_tile(j), t_end - 1);
            const int key = min(t * 32 + ld_row(j), kv_len - 1);
            const u32x4 *kp = reinterpret_cast<const u32x4 *>(kbase + (int64_t)key * D + ld_col * 8);
            const u32x4 *vp = reinterpret_cast<const u32x4 *>(vbase + (int64_t)key * D + ld_col * 8);
            if constexpr (ONCE) {
                kr[j] = __builtin_nontemporal_load(kp);
                vr[j] = __builtin_nontemporal_load(vp);
            } else {
                kr[j] = *kp;
                vr[j] = *vp;
            }
        }
    };
    if (n_my > 0) {
#pragma unroll
        for (int pf = 0; pf < PFD; pf++)
            load_step(pf, kreg[pf], vreg[pf]);
    }

    // ---- this wave's queries: fragments, owning rows, masks
    bf16x8 qf[QG][NKS];
    int q_node_of[QG];
    bool q_valid[QG];
    bool wave_active = false;
#pragma unroll
    for (int qt = 0; qt < QG; qt++) {
        RowOwner ro = row_owner(a, kvh, qg, wave, QG, qt, c, QW);
        q_valid[qt] = ro.row >= 0;
        wave_active = wave_active || q_valid[qt];
        const int row = q_valid[qt] ? ro.row : 0;
        const int head = q_valid[qt] ? ro.head : kvh * a.group;
        q_node_of[qt] = a.q_node ? min(max(a.q_node[(int64_t)b * a.n_q + row], 0), a.n_tree - 1) : row;
        const uint16_t *qp = reinterpret_cast<const uint16_t *>(a.q) + (((int64_t)b * a.n_q + row) * a.n_q_heads + head) * D + g * 8;
#pragma unroll
        for (int ks = 0; ks < NKS; ks++)
            qf[qt][ks] = *reinterpret_cast<const bf16x8 *>(qp + ks * 32);
    }
    wave_active = __any(wave_active);
    if (!a.tree_mask && tid < a.n_tree)
        lds_parent[tid] = my_parent < tid ? my_parent : -1;   // a walk up the tree always ends
    __syncthreads();   // parents staged

    NodeMask<MW> qmask[QG];
#pragma unroll
    for (int qt = 0; qt < QG; qt++) {
        qmask[qt] = q_valid[qt] ? visible_nodes<MW>(a, b, q_node_of[qt], lds_parent) : empty_mask<MW>();
        if (!q_valid[qt]) {
#pragma unroll
            for (int ks = 0; ks < NKS; ks++)
#pragma unroll
                for (int i = 0; i < 8; i++)
                    qf[qt][ks][i] = (__bf16)0.0f;
        }
    }

    WaveState<QG, NDT> st;
#pragma unroll
    for (int qt = 0; qt < QG; qt++) {
        st.m[qt] = -INFINITY;
        st.l[qt] = 0.0f;
#pragma unroll
        for (int dt = 0; dt < NDT; dt++)
            st.o[qt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // one step of KT tiles: registers -> LDS stage, barrier, refill the register set, compute from LDS
    auto step = [&](int i, u32x4(&kr)[NLD], u32x4(&vr)[NLD]) {
        uint16_t *stage = lds + (i & 1) * GS::STAGE_ELEMS;
#pragma unroll
        for (int j = 0; j < NLD; j++) {
            uint16_t *tile = stage + ld_tile(j) * G::TILE_ELEMS;
            *reinterpret_cast<u32x4 *>(tile + ld_row(j) * KSTR + ld_col * 8) = kr[j];
            *reinterpret_cast<u32x4 *>(tile + 32 * KSTR + ld_row(j) * VSTR + ld_col * 8) = vr[j];
        }
        __syncthreads();
        load_step(i + PFD, kr, vr);
        if (!wave_active)
            return;
        tiles_compute<D, QG, KT, MW>(stage + kgrp * KT * G::TILE_ELEMS, (t_begin + (i * KG + kgrp) * KT) * 32, P, key_end, a.n_tree, a.scale_log2, qf,
                                        qmask, st, c, g);
    };

    // every load issued so far (queries, masks, first tiles) has to land before the loop: the in-order
    // load counter then only ever counts tile prefetches inside it
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    {
        int i = 0;
        for (; i + PFD <= n_steps; i += PFD) {
#pragma unroll
            for (int pf = 0; pf < PFD; pf++)
                step(i + pf, kreg[pf], vreg[pf]);
        }
        // leftover steps run outside the loop so that its body always issues the same number of loads
#pragma unroll
        for (int pf = 0; pf < PFD - 1; pf++)
            if (i + pf < n_steps)
                step(i + pf, kreg[pf], vreg[pf]);
    }
    __syncthreads();   // every wave is done with the last tile: the stage areas can be reused for states and output rows
    constexpr int STATE = StateGeom<D, QG>::STATE_FLOATS;
    if (KG == 2) {
        // the second key group parks its states; the first adds them to its own (a barrier in between, so no early exit)
        float *sbuf = reinterpret_cast<float *>(smem_raw) + wave * STATE;
        if (kgrp == 1 && wave_active)
            state_store<QG, NDT>(st, sbuf, lane);
        __syncthreads();
        if (kgrp == 1 || !wave_active)
            return;
        state_merge<QG, NDT>(st, sbuf, lane);
    }
    if (!wave_active)
        return;

    // the softmax sum was kept per lane over the lane's own key rows: complete it across the 4 row groups
#pragma unroll
    for (int qt = 0; qt < QG; qt++) {
        float l = st.l[qt];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        st.l[qt] = l;
    }
    if (NW == 4 && nsplit > 1) {
        // several splits: publish this wave's state for attn_merge_kernel (the launch plan never splits the 8-wave form)
        const int64_t grp = ((int64_t)b * a.n_kv_heads + kvh) * a.n_qg + qg;
        state_store<QG, NDT>(st, a.part + ((grp * nsplit + split) * 4 + wave) * StateGeom<D, QG>::STATE_FLOATS, lane);
        return;
    }
    // Output rows leave through LDS: a lane holds 4 columns of one row per column tile, which stored directly would
    // be 32-byte pieces of 16 rows per instruction; staged in the wave's own LDS area (free by now) the rows go out
    // as whole 16-byte-per-lane rows, full cache lines per instruction, with the nontemporal hint (nobody in this
    // launch reads them; measured together with the staging: 82.5 -> 78 us at 32 LLaVA sequences, either alone nothing).
    constexpr float LN2 = 0.6931471805599453f;
    constexpr int OSTR = D + 8, RPP = 64 / LPR;   // staging row stride; rows per store instruction (LPR lanes per row)
    constexpr size_t OT_BASE = KG == 2 ? (size_t)QW * STATE * sizeof(float) : 0;   // behind the parked states, which may still be read
    static_assert(OT_BASE + (size_t)QW * 16 * OSTR * 2 <= (size_t)2 * GS::STAGE_ELEMS * 2, "states and output staging reuse the tile stages");
    uint16_t *ot = reinterpret_cast<uint16_t *>(smem_raw + OT_BASE) + wave * 16 * OSTR;
#pragma unroll
    for (int qt = 0; qt < QG; qt++) {
        RowOwner ro = row_owner(a, kvh, qg, wave, QG, qt, c, QW);
        const float l = st.l[qt];
        const float inv = l > 0.0f ? 1.0f / l : 0.0f;
#pragma unroll
        for (int dt = 0; dt < NDT; dt++) {
            bf16x4 ob;
#pragma unroll
            for (int r = 0; r < 4; r++)
                ob[r] = (__bf16)(st.o[qt][dt][r] * inv);
            *reinterpret_cast<bf16x4 *>(ot + c * OSTR + dt * 16 + g * 4) = ob;
        }
        if (ro.row >= 0 && a.lse && g == 0)
            a.lse[((int64_t)b * a.n_q_heads + ro.head) * a.n_q + ro.row] = l > 0.0f ? (st.m[qt] + log2f(l)) * LN2 : -INFINITY;
        wave_lds_fence();
#pragma unroll
        for (int pass = 0; pass < 16 / RPP; pass++) {
            const int r2 = pass * RPP + lane / LPR, col = (lane % LPR) * 8;
            RowOwner ro2 = row_owner(a, kvh, qg, wave, QG, qt, r2, QW);
            if (ro2.row >= 0) {
                uint16_t *op = reinterpret_cast<uint16_t *>(a.out) + (((int64_t)b * a.n_q + ro2.row) * a.n_q_heads + ro2.head) * D + col;
                __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(ot + r2 * OSTR + col), reinterpret_cast<u32x4_any *>(op));
            }
        }
        wave_lds_fence();
    }
}

// s <- s (+) state at src, the associative merge of two online-softmax states
template <int QG, int NDT>
__device__ __forceinline__ void state_merge(WaveState<QG, NDT> &s, const float *src, int lane)
{
#pragma unroll
    for (int qt = 0; qt < QG; qt++) {
        float mo = src[QG * NDT * 256 + (qt * 2) * 64 + lane];
        float lo = src[QG * NDT * 256 + (qt * 2 + 1) * 64 + lane];
        float mn = fmaxf(s.m[qt], mo);
        float ms = (mn == -INFINITY) ? 0.0f : mn;
        float a1 = __builtin_amdgcn_exp2f(s.m[qt] - ms), a2 = __builtin_amdgcn_exp2f(mo - ms);
        s.l[qt] = s.l[qt] * a1 + lo * a2;
        s.m[qt] = mn;
#pragma unroll
        for (int dt = 0; dt < NDT; dt++) {
            f32x4 oo = reinterpret_cast<const f32x4 *>(src)[(qt * NDT + dt) * 64 + lane];
            s.o[qt][dt] = s.o[qt][dt] * a1 + oo * a2;
        }
    }
}

// Merge the split states of one (group, wave, query tile) in split order and write the rows.  One
// workgroup of 4 waves per state; wave w owns the 16-wide output column tiles w, w+4, ...; loads of
// up to 8 splits are in flight at once.
template <int D, int QG>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a)
{
    constexpr int NDT = D / 16, NDW = NDT / 4;
    constexpr int STATE = StateGeom<D, QG>::STATE_FLOATS;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int qt = blockIdx.x % QG;
    const int wave = (blockIdx.x / QG) % 4;
    const int64_t grp = blockIdx.x / (QG * 4);
    const int qg = (int)(grp % a.n_qg);
    const int kvh = (int)((grp / a.n_qg) % a.n_kv_heads), b = (int)(grp / ((int64_t)a.n_qg * a.n_kv_heads));
    RowOwner ro = row_owner(a, kvh, qg, wave, QG, qt, lane & 15);
    if (__all(ro.row < 0))
        return;
    const int nsplit = a.n_splits;
    const float *base = a.part + (grp * nsplit * 4 + wave) * STATE;
    const int64_t stride = (int64_t)4 * STATE;
    const int ml = QG * NDT * 256 + (qt * 2) * 64 + lane;
    float m = -INFINITY;
    for (int s0 = 0; s0 < nsplit; s0 += 8) {
        float mm[8];
#pragma unroll
        for (int j = 0; j < 8; j++)
            mm[j] = s0 + j < nsplit ? base[(s0 + j) * stride + ml] : -INFINITY;
#pragma unroll
        for (int j = 0; j < 8; j++)
            m = fmaxf(m, mm[j]);
    }
    const float ms = (m == -INFINITY) ? 0.0f : m;
    float l = 0.0f;
    f32x4 o[NDW];
#pragma unroll
    for (int d = 0; d < NDW; d++)
        o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < nsplit; s0 += 8) {
        float mm[8], ll[8];
        f32x4 oo[8][NDW];
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const bool live = s0 + j < nsplit;
            const float *src = base + (live ? s0 + j : s0) * stride;
            mm[j] = live ? src[ml] : -INFINITY;
            ll[j] = src[ml + 64];
#pragma unroll
            for (int d = 0; d < NDW; d++)
                oo[j][d] = reinterpret_cast<const f32x4 *>(src)[(qt * NDT + w + 4 * d) * 64 + lane];
        }
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const float wgt = __builtin_amdgcn_exp2f(mm[j] - ms);   // 0 for splits past the end
            l += wgt * ll[j];
#pragma unroll
            for (int d = 0; d < NDW; d++)
                o[d] += oo[j][d] * wgt;
        }
    }
    if (ro.row < 0)
        return;
    const int g = lane >> 4;
    const float inv = l > 0.0f ? 1.0f / l : 0.0f;
    uint16_t *op = reinterpret_cast<uint16_t *>(a.out) + (((int64_t)b * a.n_q + ro.row) * a.n_q_heads + ro.head) * D + g * 4;
#pragma unroll
    for (int d = 0; d < NDW; d++) {
        bf16x4 ob;
#pragma unroll
        for (int r = 0; r < 4; r++)
            ob[r] = (__bf16)(o[d][r] * inv);
        *reinterpret_cast<u32x2_any *>(op + (w + 4 * d) * 16) = __builtin_bit_cast(u32x2_any, ob);
    }
    if (a.lse && g == 0 && w == 0)
        a.lse[((int64_t)b * a.n_q_heads + ro.head) * a.n_q + ro.row] = l > 0.0f ? (m + log2f(l)) * 0.6931471805599453f : -INFINITY;
}

// A few query tiles for one key stream (attn_wave_kernel, attn_pair_kernel, attn_quad_kernel).  A workgroup serves QS * QT query tiles of one KV head and one
// slice of DV = D / DS output columns; its QS * KG waves are KG key groups, which take the KEYS-key tiles of the range in turn, times QS
// query slots of QT tiles.  The key groups' states meet in LDS once, at the end.  The rows that share a KV head are numbered through
// all heads of the group (row f is row f % n_q of head f / n_q), so only a KV head's last tile can be partly empty: 33 rows of 2 heads
// are 5 tiles, not 6.
//
// What bounds such a launch is what a CU can pull: 60 to 75 GB/s whatever is in flight and however it is loaded (nothing but loads: 256
// workgroups of 672 KB, four to a stream, 14.1 us; 8 to a stream of 1344 KB, 21.7 us), then the chain ahead of the first tile and
// behind the last one.  So the work that goes with the bytes stays out of their way:
// - Tiles go from memory straight to LDS, with no staging registers, no LDS write instructions and no barrier in the loop: with one slot
//   a wave has its own tiles (K of the tile after next is requested when this tile's scores are formed, V of the next one when this
//   tile's product is), with two the slots of a group share them, one loading K and one V into the stage that is free, and meet once a
//   step; with four, two load K and two V, into a ring of four stages.  The groups drift apart, so that some waves are in their exponentials while others are in their MFMAs (a barrier per step
//   instead of the meeting: 14.6 us for the loop below instead of 11.2).
// - A fragment read from LDS serves QT MFMAs; with one query tile per wave the LDS reads alone took half the time of such a kernel.  Four
//   tiles in every wave need no slots, but twice the states to merge: 3.6 us of 20 at head_dim 128, against 2.2 with two slots.
// - 8 query tiles take four slots: as long as that leaves one workgroup per CU, two with 4 tiles each on a CU pull the keys twice, one
//   after the other.  There the MFMAs and exponentials of a step (0.9 us of the 1.3 it takes) bound the launch, no longer the pull.
// - With DS slices the scores are formed DS times, but K and 1 / DS of V is all a workgroup pulls, and the states are small.
// Measured per launch, the kernels these replaced / here: 32 heads x 764 keys x 60 rows 10.0 / 8.9 us; 4 sequences x 8 KV heads x up to 1316
// keys x 33 rows of 2 heads, head_dim 256, 27.3 / 20.6 us; 8 sequences x 8 KV heads x up to 1340 keys x 60 rows of 4 heads 23.2 / 20.8 us
// (start to scores 3 us, loop 11, states and rows 2.3); 16 sequences of that, in four slots, 40.6 / 33.5 us.
//
// The 16-byte pieces of a tile's rows lie swapped (lds_tiles.h), so that neither the 16-byte reads of K nor the
// transposing reads of V meet in a bank.  The loads need 16-byte aligned tensors: others take attn_bf16_kernel.
template <int D, int DS, int QT, int QS, int KG, int KEYS>
struct RowsGeom {
    static constexpr int DV = D / DS, KROW = D * 2, VROW = DV * 2, NW = QS * KG;   // bytes of a K row, of a V slice's row; waves
    static constexpr int STEP_KEYS = KG * KEYS;                                    // keys of a step of all key groups
    static constexpr int KTILE = KEYS * KROW, VTILE = KEYS * VROW, NK = KTILE / 1024, NV = VTILE / 1024;   // bytes and 16-byte loads per lane of a tile
    static constexpr int NDT = DV / 16, NKS = D / 32, NH = KEYS / 16;              // column tiles, key steps, 16-key halves
    static constexpr int UNIT = QT * NDT * 1024, QTILE = 16 * KROW;                // bytes of a wave's outputs, of a query tile
    // LDS: the tiles of the key groups (K, V and a second K stage, with two query slots a second V stage as well), whose place the waves'
    // outputs take at the end; references and sums; every wave's masks; parents; the slots' step counts.  The queries lie where they fit:
    // with one slot tile i where group i's second K stage will be, with two behind the stages of the groups or of all, with four where the last
    // stages will be, filled when the queries are in registers
    static constexpr int GROUP = KTILE + VTILE, NS = QS == 4 ? 4 : 2, STAGES = QS > 1 ? NS * GROUP : GROUP + KTILE, STRIDE = STAGES > QS * UNIT ? STAGES : QS * UNIT, TILES = KG * STRIDE;
    static constexpr bool Q_APART = QS == 2 && STRIDE - STAGES < QTILE;
    static constexpr int Q_PER = QS == 4 ? QS * QT / KG : 1;                       // query tiles that lie together
    static constexpr int EARLY = QS == 4 ? (STRIDE - Q_PER * QTILE) / GROUP : NS;  // stages that hold no queries
    static constexpr int Q_OFF = Q_APART ? TILES : QS > 1 ? EARLY * GROUP : GROUP, Q_STRIDE = Q_APART ? QTILE : STRIDE;
    static constexpr int q_at(int i) { return Q_OFF + i / Q_PER * Q_STRIDE + i % Q_PER * QTILE; }
    // Odd workgroups of a KV head take the tiles of every two steps in the other order: half of what a workgroup reads has then come to L2 for another one, and from there a CU
    // pulls twice as fast (138 against 70 GB/s).  (In lock step it asks for lines that are still on their way; L2 counts those as hits too.)  That pays while the keys and values which an XCD's heads have in flight stay in L2: 32 heads of 64 in two
    // slices, 1660 keys 9.9 -> 9.3 us, 2260 keys 12.4 -> 11.5, up to 560 keys equal.  Elsewhere sharing a miss in lock step is better: two tiles unsliced
    // at 4 sequences 13.3 -> 16.6, pairs at 8 sequences 20.3 -> 21.0; four slices 1 % either way.  The hint undoes it, so these kernels read without
    // (10.0 with both).  With the keys still in the memory-side cache, as between the levels of a draft, the same within 1 % (7.38 / 7.45), the first
    // level 11.2 -> 10.2.
    static constexpr bool SWAPPED = QS == 1 && D == 64 && DS == 2;
    // The same with more steps and workgroups: of every TURN steps behind the first, which all take together (the first scores come as early), the workgroups of a KV head start
    // with another one each and go round, so that most of what they read has come to L2 before they ask for it: a read request of a CU takes 390 clocks instead of 552 (one LLaVA sequence, 60 rows),
    // 465 instead of 555 (four Gemma3 sequences of 33), while L2 counts as many hits and misses either way (0.83 and 0.79 of the requests hit).  For launches where the pull is far longer than the MFMAs and exponentials beside it: one
    // query tile, or head_dim 256 in slices.  Nothing but the loads, 1 sequence of 8 KV heads, 60 rows of 4 heads, 1340 keys: 11.5 us, with the order 9.1; the launch 11.7 and 10.4.
    // TURN 2, 4, 8, 16 there: 11.2, 11.0, 10.7, 10.7, with the first step turned too 0.1 us more each; which workgroups take it: see order_of_tiles().
    static constexpr bool TURNED = QS == 1 && !SWAPPED && (QT == 1 || D == 256);
    static constexpr int LOADERS = QS == 4 ? 2 : 1;                                // waves that share the loads of a K tile, and of a V tile
    static constexpr int ML_OFF = TILES + (Q_APART ? QS * QT * QTILE : 0), MASK_OFF = ML_OFF + NW * QT * 32 * 4, PAR_OFF = MASK_OFF + NW * QT * 16 * 8, MEET_OFF = PAR_OFF + 64 * 4;
    static constexpr size_t BYTES = MEET_OFF + NW * 4;
    static_assert(BYTES <= 160 * 1024 && (Q_APART || QS * QT <= KG * Q_PER) && (QS > 1 || QTILE <= KTILE) && EARLY >= 1 && EARLY <= NS, "a workgroup's LDS");
};

// What a workgroup needs ahead of its first loads, as plain arguments: the 14 dwords that are in scalar registers when a wave starts (a structure is read from memory).  The
// plan's limits make them fit: at most 256 streams of up to 4 query heads, 256 rows, s_max below 2^24.  What comes behind them is asked for together with the prefix length.
// us a launch, all arguments from a structure in two batches / in one / so: one LLaVA sequence 8.71 / 8.46 / 8.36, 30 rows of it 8.42 / 8.15 / 7.99, two Gemma3 sequences of 33 rows 16.9 / 16.6 / 16.3 (with RowsGeom::TURNED).
struct RowsHead {
    const int32_t *prefix_len;
    const void *q, *k;
    const int32_t *parent;   // null: there is a mask
    uint32_t heads, rows;    // n_kv_heads + 2^16 * group, n_q + 2^16 * n_tree
    uint32_t spread, nq_magic, s_max, n_streams;
};
#define ROWS_PARAMETERS const int32_t *prefix_len, const void *q, const void *k, const int32_t *parent, uint32_t heads, uint32_t rows, uint32_t spread, uint32_t nq_magic, uint32_t s_max, uint32_t n_streams, AttnArgs rest
#define ROWS_ARGUMENTS with_head(rest, {prefix_len, q, k, parent, heads, rows, spread, nq_magic, s_max, n_streams})
__device__ __forceinline__ AttnArgs with_head(const AttnArgs &rest, const RowsHead &h)
{
    AttnArgs a = rest;
    a.prefix_len = h.prefix_len;
    a.q = h.q; a.k = h.k; a.parent = h.parent;
    a.n_kv_heads = (int)(h.heads & 0xffff);
    a.group = (int)(h.heads >> 16);
    a.n_q_heads = a.n_kv_heads * a.group;
    a.n_q = (int)(h.rows & 0xffff);
    a.n_tree = (int)(h.rows >> 16);
    a.spread = h.spread;
    a.nq_magic = h.nq_magic;
    a.s_max = h.s_max;
    a.n_streams = (int)h.n_streams;
    return a;
}

// How a launch reads its tiles, each a form of the kernel of its own: in the order of the keys, the same with the nontemporal hint (AttnArgs::once), in turned order
// (RowsGeom::TURNED, AttnArgs::turn), or in the order of the keys with nothing asked for before it is known how many there are (short_range()).  (With the turn a number that may be zero, every step of a launch in the order of the keys worked out its place for nothing: drafting, 10 rows of 32 on 8 heads of 128,
// 4 sequences of 1283 keys 9.7 us, 9.2 so, 900 keys 8.2 and 7.9.)
enum { READ_PLAIN, READ_ONCE, READ_TURNED, READ_SHORT };

template <int N>
__device__ __forceinline__ void wait_loads()   // until at most N of this wave's loads are in flight
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// x / d for x * d below 2^32: magic = ceil(2^32 / d), or 0 for d = 1
__device__ __forceinline__ int quick_div(int x, uint32_t magic) { return magic ? (int)__umulhi((uint32_t)x, magic) : x; }

// The SLOTS adjacent waves of a key group wait for each other: each writes how often it has been here and reads the others' counts until they
// have come as far.  The LDS operations of a wave take effect in order, so what a wave wrote or read before, the others find done.
template <int SLOTS>
__device__ __forceinline__ void slots_meet(uint32_t meet, int wave, int count)
{
    typedef __attribute__((address_space(3))) volatile int lds_int;
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) volatile i32x4 lds_int4;
    asm volatile("" ::: "memory");
    *(lds_int *)(uintptr_t)(meet + 4 * wave) = count;
    if constexpr (SLOTS == 2) {
        while (__builtin_amdgcn_readfirstlane(*(lds_int *)(uintptr_t)(meet + 4 * (wave ^ 1))) < count)
            ;
    } else {
        static_assert(SLOTS == 4, "a key group's counts are read together");
        for (;;) {
            const i32x4 at = *(lds_int4 *)(uintptr_t)(meet + 4 * (wave & ~3));
            if (__builtin_amdgcn_readfirstlane(min(min(at[0], at[1]), min(at[2], at[3]))) >= count)
                break;
        }
    }
    asm volatile("" ::: "memory");
}

template <int D, int DS, int QT, int QS, int KG, int KEYS, int FORM>
__device__ __forceinline__ void attend_rows(const AttnArgs &a)
{
    using G = RowsGeom<D, DS, QT, QS, KG, KEYS>;
    constexpr bool ONCE = FORM == READ_ONCE, TURNED = FORM == READ_TURNED;
    static_assert(!TURNED || G::TURNED, "a form of its own for the order that this geometry has");
    constexpr int KROW = G::KROW, VROW = G::VROW, NW = G::NW, NDT = G::NDT, NKS = G::NKS, NH = G::NH, NK = G::NK, NV = G::NV, TILES_Q = QS * QT;
    constexpr int LPK = KROW / 16, LPV = VROW / 16;                // lanes per row of a load
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), qs = wave % QS, kg = wave / QS;
    const int c = lane & 15, g = lane >> 4;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem_raw;

    // workgroups of a KV head have ids congruent mod 8 (same XCD).  The KV heads of all sequences take the XCDs in turn: 4 or 5 heads numbered
    // per sequence left XCDs idle (24 sequences of 4 KV heads, 33 rows of 4 heads, 340 keys: 27.1 us, 15.0 in turn)
    int kvh = blockIdx.y * 8 + (blockIdx.x & 7), b = blockIdx.z;
    const int unit = blockIdx.x >> 3, ds = unit % DS;
    if (__builtin_expect(a.spread != 0, 0)) {
        const int stream = kvh;
        b = (int)((stream * a.spread) >> 16);          // exact: fewer than 264 streams
        kvh = stream < a.n_streams ? stream - b * a.n_kv_heads : a.n_kv_heads;
    }
    const int n_rows = a.group * a.n_q, row0 = unit / DS * (TILES_Q * 16);
    if (kvh >= a.n_kv_heads || row0 >= n_rows)
        return;
    const int prefix = a.prefix_len[b];   // (ahead of the first asm statement, so that it stays a scalar load)

    // ---- the queries and the parents, straight to LDS (rows past the last one: the last one again; they are never stored)
    {
        const uint16_t *qb = reinterpret_cast<const uint16_t *>(a.q) + ((int64_t)b * a.n_q * a.n_q_heads + (int64_t)kvh * a.group) * D;
        for (int i = wave; i < TILES_Q * 16 * KROW / 1024; i += NW) {
            const int r = i * (64 / LPK) + lane / LPK;             // row of the workgroup
            const int f = min(row0 + r, n_rows - 1), hh = quick_div(f, a.nq_magic), row = f - hh * a.n_q;
            lds_load16(qb, (uint32_t)((row * a.n_q_heads + hh) * KROW + (((lane % LPK) ^ (D == 64 ? (r >> 1) & 7 : r & 15)) * 16)), lds0 + G::q_at(i / (G::QTILE / 1024)) + i % (G::QTILE / 1024) * 1024);
        }
        if (wave == NW - 1 && a.parent)
            lds_load4(a.parent + (int64_t)b * a.n_tree, (uint32_t)min(lane, a.n_tree - 1) * 4, lds0 + G::PAR_OFF);
    }

    // ---- tile loads: a lane's 16 bytes of instruction j go to 1024 * j + 16 * lane of the tile's area
    const unsigned char *kbase = reinterpret_cast<const unsigned char *>(a.k) + ((int64_t)b * a.n_kv_heads + kvh) * a.s_max * KROW;
    const unsigned char *vbase = reinterpret_cast<const unsigned char *>(a.v) + ((int64_t)b * a.n_kv_heads + kvh) * a.s_max * KROW + ds * VROW;
    // (two loaders of a tile take a half of its instructions each: the second's rows lie k_half, v_half rows on, and the half's number is a bit of
    // its own in the swizzle)
    auto scalar = [](uint32_t x) { return G::LOADERS == 2 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)x) : x; };   // (the same in every lane; the compiler puts the half in a vector register)
    constexpr int KJ = NK / G::LOADERS, VJ = NV / G::LOADERS;
    static_assert(G::LOADERS == 1 || ((swizzle_k<KROW>(KJ) & swizzle_k<KROW>(KJ - 1)) == 0 && (swizzle_v<VROW>(VJ) & swizzle_v<VROW>(VJ - 1)) == 0), "loaders");
    const int half = G::LOADERS == 2 ? qs & 1 : 0, k_half = half * (KJ * (64 / LPK)), v_half = half * (VJ * (64 / LPV));
    const int krow = lane / LPK, vrow = lane / LPV;
    const int kl = piece_k<KROW>(lane) ^ (half * swizzle_k<KROW>(KJ)), vl = piece_v<VROW>(lane) ^ (half * swizzle_v<VROW>(VJ));
    // (`rows`: the live ones, or those of the cache)
    auto issue_k = [&](int t, int at, int rows) {
        const uint32_t dst = scalar(lds0 + at + half * (KJ * 1024));
        if ((t + 1) * KEYS <= rows) {
            const unsigned char *p = kbase + (int64_t)t * (KEYS * KROW) + k_half * KROW;
#pragma unroll
            for (int j = 0; j < KJ; j++)
                lds_load16<ONCE>(p + j * 1024, (uint32_t)(krow * KROW + (kl ^ swizzle_k<KROW>(j))), dst + j * 1024);
        } else {
            // the ragged end: rows past the last live one are that one again (their scores are masked)
#pragma unroll
            for (int j = 0; j < KJ; j++)
                lds_load16(kbase, (uint32_t)(min(t * KEYS + k_half + j * (64 / LPK) + krow, rows - 1) * KROW + (kl ^ swizzle_k<KROW>(j))), dst + j * 1024);
        }
    };
    // Every wave's first keys are asked for before it is known how many there are: any row of the cache may be read, whatever it holds, and a score behind the last live one is masked (a value is
    // multiplied with its zero, so those wait).  us a launch, behind the prefix length / ahead of it: one LLaVA sequence 8.36 / 8.14, 250 keys 5.94 / 5.73, one Gemma3 sequence 15.25 / 14.99,
    // twelve 27.9 / 27.9.  Not in short ranges: see short_range().
    // (With 1 << 30 rows, which leaves the compiler no branch here, one LLaVA sequence 8.37 instead of 8.18: the other arguments are then asked for ahead of these loads.)
    constexpr bool FIRST = !G::SWAPPED && FORM != READ_SHORT;
    const bool first_mine = FIRST && (QS == 1 || qs < QS / 2);
    if (first_mine)
        issue_k(kg, kg * G::STRIDE, (int)a.s_max);

    // All other arguments, in the same trip to memory as the prefix length: those that stand behind the barrier below were asked for there, one or two trips ahead of the first scores.  us a launch,
    // there / here: one LLaVA sequence 8.54 / 8.41, 1400 keys 11.9 / 11.5, two of 704 keys 10.4 / 10.1, four of 33 rows 11.6 / 11.2, four Gemma3 sequences of 33 rows 18.9 / 18.6, eight Pixtral ones 19.4 / 18.9.
    asm volatile("" ::"s"(a.v), "s"(a.q_node), "s"(a.tree_mask), "s"(a.out), "s"(a.lse), "s"(a.include_self), "s"(a.turn), "s"(a.scale_log2));
    const int P = (int)min((int64_t)max(prefix, 0), a.s_max - a.n_tree);   // never past the cache, whatever the array holds
    const int kv_len = P + a.n_tree;
    const int t_end = (kv_len + KEYS - 1) / KEYS;

    auto issue_v = [&](int t, int at) {
        const uint32_t dst = scalar(lds0 + at + half * (VJ * 1024));
        if ((t + 1) * KEYS <= kv_len) {
            const unsigned char *p = vbase + (int64_t)t * (KEYS * KROW) + v_half * KROW;
#pragma unroll
            for (int j = 0; j < VJ; j++)
                lds_load16<ONCE>(p + j * (64 / LPV) * KROW, (uint32_t)(vrow * KROW + (vl ^ swizzle_v<VROW>(j))), dst + j * 1024);
        } else {
#pragma unroll
            for (int j = 0; j < VJ; j++)
                lds_load16(vbase, (uint32_t)(min(t * KEYS + v_half + j * (64 / LPV) + vrow, kv_len - 1) * KROW + (vl ^ swizzle_v<VROW>(j))), dst + j * 1024);
        }
    };
    // one query slot: a wave's own K, V and second K areas.  Two and four: the key group's, stage by stage; the lower half of the slots loads its K
    // tiles, the upper half its V tiles
    int ktile = kg * G::STRIDE;
    [[maybe_unused]] int ktile2 = ktile + G::GROUP;
    const int vtile = ktile + G::KTILE;
    int t = kg;
    auto wait_slot = [&](auto n) {      // until the loads of at most n steps are in flight
        if (qs < QS / 2)
            wait_loads<n * KJ>();
        else
            wait_loads<n * VJ>();
    };
    auto wait_steps = [&](int n) {
        if (n <= 0)
            wait_loads<0>();
        else if (n == 1)
            wait_slot(std::integral_constant<int, 1>());
        else if (n == 2 || G::NS == 2)
            wait_slot(std::integral_constant<int, 2>());
        else
            wait_slot(std::integral_constant<int, G::NS == 2 ? 2 : 3>());
    };
    auto issue_slot = [&](int t, int at) {
        if (qs < QS / 2)
            issue_k(t, at, kv_len);
        else
            issue_v(t, at + G::KTILE);
    };
    const int n_steps = (max(t_end - kg, 0) + KG - 1) / KG;
    const int odd = G::SWAPPED && a.turn ? unit & 1 : 0, turned = TURNED ? (int)((unit * a.turn) >> 16) : 0;
    auto tile = [&](int i) {                  // the key tile of this wave's step i
        if (G::SWAPPED)
            i = (i | 1) < n_steps ? i ^ odd : i;
        return kg + KG * (TURNED ? turned_step(i, n_steps, turned) : i);
    };
    const bool early = QS == 1 && kg >= QT;   // the second K stage holds no queries
    const uint32_t meet = lds0 + G::MEET_OFF;
    if (QS > 1)
        *reinterpret_cast<int *>(smem_raw + G::MEET_OFF + 4 * wave) = 0;
    if (t < t_end) {
        if constexpr (QS > 1) {
#pragma unroll
            for (int i = 0; i < G::EARLY; i++)
                if (i < n_steps && (i > 0 || !first_mine))
                    issue_slot(t + i * KG, ktile + i * G::GROUP);
            wait_steps(min(n_steps, G::EARLY));   // the queries and parents are there; the first tiles stay in flight
        } else {
            if (!FIRST)
                issue_k(tile(0), ktile, kv_len);
            issue_v(tile(0), vtile);
            if (early && n_steps > 1) {
                issue_k(tile(1), ktile2, kv_len);
                wait_loads<2 * NK + NV>();
            } else {
                wait_loads<NK + NV>();
            }
        }
    } else if (first_mine) {
        wait_loads<KJ>();               // (a wave without keys: what it asked for all the same is waited for ahead of the states)
    } else {
        wait_loads<0>();
    }
    __syncthreads();
    // ---- query fragments
    bf16x8 qf[QT][NKS];
    const int foff = fragment_k<KROW>(c, g);
#pragma unroll
    for (int qt = 0; qt < QT; qt++)
#pragma unroll
        for (int ks = 0; ks < NKS; ks++)
            qf[qt][ks] = *reinterpret_cast<const bf16x8 *>(smem_raw + G::q_at(qs * QT + qt) + at_key_step(foff, ks));
    if constexpr (!G::Q_APART)
        __syncthreads();                // every wave has its queries
    if constexpr (QS == 1) {
        if (!early && n_steps > 1)
            issue_k(tile(1), ktile2, kv_len);
    } else {
#pragma unroll
        for (int i = G::EARLY; i < G::NS; i++)
            if (i < n_steps)
                issue_slot(t + i * KG, ktile + i * G::GROUP);
    }
    // ---- what the wave's rows see of the tree: lanes 16 * qt .. work out query tile qt's
    uint64_t *masks = reinterpret_cast<uint64_t *>(smem_raw + G::MASK_OFF) + wave * QT * 16;
    if (g < QT) {
        const int f = row0 + (qs * QT + g) * 16 + c;
        uint64_t mk = 0ull;
        if (f < n_rows) {
            const int row = f - quick_div(f, a.nq_magic) * a.n_q;
            const int node = a.q_node ? min(max(a.q_node[(int64_t)b * a.n_q + row], 0), a.n_tree - 1) : row;
            if (a.tree_mask) {
                mk = a.tree_mask[(int64_t)b * a.n_tree + node] & (~0ull >> (64 - a.n_tree));
            } else {
                const int32_t *par = reinterpret_cast<const int32_t *>(smem_raw + G::PAR_OFF);
                if (a.include_self)
                    mk = 1ull << node;
                for (int p = node, q = par[p]; q >= 0 && q < p; p = q, q = par[p])   // (a parent that does not precede its node is none)
                    mk |= 1ull << q;
            }
        }
        masks[lane] = mk;
    }
    wave_lds_fence();

    f32x4 o[QT][NDT];
    float m[QT], l[QT];
#pragma unroll
    for (int qt = 0; qt < QT; qt++) {
        m[qt] = -INFINITY;
        l[qt] = 0.0f;
#pragma unroll
        for (int dt = 0; dt < NDT; dt++)
            o[qt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int voff = fragment_v<VROW>(c, g);
    const float scale_log2 = a.scale_log2;

    // S^T = K Q^T of the tile at `at`: its fragments are all requested first
    auto scores = [&](int at, f32x4(&s)[NH][QT]) {
        bf16x8 kf[NKS][NH];
#pragma unroll
        for (int ks = 0; ks < NKS; ks++)
#pragma unroll
            for (int h = 0; h < NH; h++)
                kf[ks][h] = *reinterpret_cast<const bf16x8 *>(smem_raw + at + h * 16 * KROW + at_key_step(foff, ks));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < NH; h++)
#pragma unroll
            for (int qt = 0; qt < QT; qt++)
                s[h][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < NKS; ks++)
#pragma unroll
            for (int h = 0; h < NH; h++)
#pragma unroll
                for (int qt = 0; qt < QT; qt++)
                    s[h][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks][h], qf[qt][ks], s[h][qt], 0, 0, 0);
    };
    // V^T fragments of column tiles dt0 .. dt0 + N - 1 of the tile at `at`
    auto read_v = [&](int at, int dt0, auto &vf) {
#pragma unroll
        for (int i = 0; i < (int)(sizeof vf / sizeof vf[0]); i++) {
            const unsigned char *vp = smem_raw + at + at_column_tile(voff, dt0 + i);
#pragma unroll
            for (int h = 0; h < NH; h++)
                vf[i][h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(vp + h * 16 * VROW));
        }
    };
    // online softmax of tile t; a column's reference is raised only when a score exceeds it by DREAM_SOFTMAX_SLACK octaves
    auto softmax = [&](int t, f32x4(&s)[NH][QT], __bf16(&p)[QT][NH * 4]) {
        const int r0 = t * KEYS - P;   // tree node of the tile's first key
        float mult = scale_log2, mx[QT];
        if (r0 + KEYS > 0 || scale_log2 < 0.0f) {
            mult = 1.0f;
#pragma unroll
            for (int qt = 0; qt < QT; qt++) {
                const uint64_t mk = masks[qt * 16 + c];
                // bit i: key i of the tile is visible (all of the prefix, what the mask says of the tree, nothing behind it)
                const uint32_t vis = (r0 <= -32 ? ~0u : r0 >= 64 ? 0u : r0 >= 0 ? (uint32_t)(mk >> r0) : (uint32_t)((mk << -r0) | ((1ull << -r0) - 1))) >> (g * 4);
                mx[qt] = -INFINITY;
#pragma unroll
                for (int e = 0; e < NH * 4; e++) {
                    const float x = (vis >> ((e >> 2) * 16 + (e & 3))) & 1u ? s[e >> 2][qt][e & 3] * scale_log2 : -INFINITY;
                    s[e >> 2][qt][e & 3] = x;
                    mx[qt] = fmaxf(mx[qt], x);
                }
            }
        } else {
#pragma unroll
            for (int qt = 0; qt < QT; qt++) {
                float x = -INFINITY;
#pragma unroll
                for (int e = 0; e < NH * 4; e++)
                    x = fmaxf(x, s[e >> 2][qt][e & 3]);
                mx[qt] = x * scale_log2;
            }
        }
        bool raise = false;
#pragma unroll
        for (int qt = 0; qt < QT; qt++)
            raise = raise || mx[qt] > m[qt] + DREAM_SOFTMAX_SLACK;
        if (__any(raise)) {
#pragma unroll
            for (int qt = 0; qt < QT; qt++) {
                float x = fmaxf(mx[qt], __shfl_xor(mx[qt], 16));
                x = fmaxf(x, __shfl_xor(x, 32));
                if (x > m[qt] + DREAM_SOFTMAX_SLACK) {
                    const float alpha = __builtin_amdgcn_exp2f(m[qt] - x);   // 0 when the old reference was -inf
                    m[qt] = x;
                    l[qt] *= alpha;
#pragma unroll
                    for (int dt = 0; dt < NDT; dt++)
                        o[qt][dt] *= alpha;
                }
            }
        }
#pragma unroll
        for (int qt = 0; qt < QT; qt++) {
            const float neg_m = m[qt] == -INFINITY ? 0.0f : -m[qt];
            float sum = 0.0f;
#pragma unroll
            for (int e = 0; e < NH * 4; e++) {
                const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e >> 2][qt][e & 3], mult, neg_m));
                sum += x;
                p[qt][e] = (__bf16)x;
            }
            l[qt] += sum;
        }
    };
    // O^T += V^T P^T for column tiles dt0 ..
    auto product = [&](int dt0, const auto &vf, const __bf16(&p)[QT][NH * 4]) {
#pragma unroll
        for (int i = 0; i < (int)(sizeof vf / sizeof vf[0]); i++)
#pragma unroll
            for (int qt = 0; qt < QT; qt++) {
                if constexpr (NH == 2) {
                    const bf16x8 v = __builtin_bit_cast(bf16x8, __builtin_shufflevector(vf[i][0], vf[i][NH - 1], 0, 1, 2, 3, 4, 5, 6, 7));
                    const bf16x8 pf = {p[qt][0], p[qt][1], p[qt][2], p[qt][3], p[qt][NH * 4 - 4], p[qt][NH * 4 - 3], p[qt][NH * 4 - 2], p[qt][NH * 4 - 1]};
                    o[qt][dt0 + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, pf, o[qt][dt0 + i], 0, 0, 0);
                } else {
                    const bf16x4 pf = {p[qt][0], p[qt][1], p[qt][2], p[qt][3]};
                    o[qt][dt0 + i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[i][0], __builtin_bit_cast(s16x4, pf), o[qt][dt0 + i], 0, 0, 0);
                }
            }
    };
    constexpr int VB = NDT / 2;         // column tiles whose V fragments are requested together
    s16x4 va[VB][NH], vb[VB][NH];
    f32x4 s[NH][QT];
    __bf16 p[QT][NH * 4];
    if constexpr (QS > 1) {
        // The waves of a key group meet at every step: each says that its share of the step's tiles is there, which also says that it is
        // done with the stage before.  (All always come: a key group's waves take the same number of steps.)
        int before = ktile + (G::NS - 1) * G::GROUP;      // the stage of the step before
        for (int i = 1; i <= n_steps; i++, t += KG) {
            if constexpr (G::NS == 2) {
                if (i == 1 && t + KG < t_end)
                    wait_slot(std::integral_constant<int, 1>());
                else
                    wait_loads<0>();
            } else {
                wait_steps(min(n_steps - i, i == 1 ? G::NS - 1 : G::NS - 2));
            }
            slots_meet<QS>(meet, wave, i);
            if (i > 1 && t + (G::NS - 1) * KG < t_end)
                issue_slot(t + (G::NS - 1) * KG, before);
            scores(ktile, s);
            read_v(ktile + G::KTILE, 0, va);
            softmax(t, s, p);
            read_v(ktile + G::KTILE, VB, vb);
            __builtin_amdgcn_sched_barrier(0);
            product(0, va, p);
            product(VB, vb, p);
            const int x = ktile;
            ktile = G::NS == 2 ? before : i % G::NS ? ktile + G::GROUP : kg * G::STRIDE;
            before = x;
        }
        wait_loads<0>();                           // (of a wave without keys)
        wait_lds();
        slots_meet<QS>(meet, wave, n_steps + 1);   // (the tiles are nobody's any more)
    } else {
        int now = tile(0), next = tile(1);
        for (int i = 0; i < n_steps; i++) {
            const bool more = i + 1 < n_steps, more2 = i + 2 < n_steps;
            const int after = tile(i + 2);
            if (more)
                wait_loads<NK + NV>();  // this tile's K (behind it: this tile's V and the next one's K)
            else
                wait_loads<NV>();
            scores(ktile, s);
            wait_lds();
            if (more2)
                issue_k(after, ktile, kv_len);
            softmax(now, s, p);
            if (more2)
                wait_loads<NK>();       // this tile's V
            else
                wait_loads<0>();
            read_v(vtile, 0, va);
            read_v(vtile, VB, vb);
            __builtin_amdgcn_sched_barrier(0);
            product(0, va, p);
            wait_lds();
            if (more)
                issue_v(next, vtile);
            product(VB, vb, p);
            now = next;
            next = after;
            const int x = ktile;
            ktile = ktile2;
            ktile2 = x;
        }
        wait_loads<0>();                           // (of a wave without keys)
    }

    // ---- the key groups' states meet: every wave leaves its outputs, references and sums where its own tiles were, and takes its share of
    // the column tiles, adding them in the order of the groups
    float *ml = reinterpret_cast<float *>(smem_raw + G::ML_OFF);      // [query tile][key group][16 references, 16 sums]
    f32x4 *xch = reinterpret_cast<f32x4 *>(smem_raw + kg * G::STRIDE + qs * G::UNIT);
#pragma unroll
    for (int qt = 0; qt < QT; qt++) {
#pragma unroll
        for (int dt = 0; dt < NDT; dt++)
            xch[(qt * NDT + dt) * 64 + lane] = o[qt][dt];
        float x = l[qt];
        x += __shfl_xor(x, 16);
        x += __shfl_xor(x, 32);
        if (g == 0) {
            ml[((qs * QT + qt) * KG + kg) * 32 + c] = m[qt];
            ml[((qs * QT + qt) * KG + kg) * 32 + 16 + c] = x;
        }
    }
    constexpr int UNITS = TILES_Q * NDT, UPW = (UNITS + NW - 1) / NW;
    static_assert(NDT % UPW == 0, "a wave's column tiles belong to one query tile");
    const int qt = wave * UPW / NDT, dt0 = wave * UPW % NDT;
    const int f = row0 + qt * 16 + c, hh = quick_div(min(f, n_rows - 1), a.nq_magic), row = f - hh * a.n_q, head = kvh * a.group + hh;
    uint16_t *op = reinterpret_cast<uint16_t *>(a.out) + (((int64_t)b * a.n_q + row) * a.n_q_heads + head) * D + ds * G::DV + dt0 * 16;
    __syncthreads();
    if (wave * UPW >= UNITS)
        return;
    float wgt[KG], mt = -INFINITY, lt = 0.0f;
#pragma unroll
    for (int k = 0; k < KG; k++) {
        wgt[k] = ml[(qt * KG + k) * 32 + c];
        mt = fmaxf(mt, wgt[k]);
    }
    f32x4 sum[UPW];
#pragma unroll
    for (int u = 0; u < UPW; u++)
        sum[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < KG; k++) {
        wgt[k] = __builtin_amdgcn_exp2f(wgt[k] - (mt == -INFINITY ? 0.0f : mt));
        lt += ml[(qt * KG + k) * 32 + 16 + c] * wgt[k];
        const f32x4 *src = reinterpret_cast<const f32x4 *>(smem_raw + k * G::STRIDE + qt / QT * G::UNIT) + ((qt % QT) * NDT + dt0) * 64 + lane;
#pragma unroll
        for (int u = 0; u < UPW; u++)
            sum[u] += src[u * 64] * wgt[k];
    }
    // The rows leave with the nontemporal hint, 64 adjacent bytes of each per instruction where a wave has two column tiles side by side: the launch is not over
    // before its rows have left the L2s.  40 launches of 8 sequences x 8 KV heads x 60 rows of 4 heads (3.9 MB of rows each), us: 32-byte pieces 821, 64-byte pieces 807, with
    // the hint 804, no rows at all 774; the same rows 40 launches later, still in the memory-side cache, 786 -> 749.  One column tile a wave: as before.
    const float inv = lt > 0.0f ? 1.0f / lt : 0.0f;
    uint2 ob[UPW];
#pragma unroll
    for (int u = 0; u < UPW; u++) {
        bf16x4 x;
#pragma unroll
        for (int r = 0; r < 4; r++)
            x[r] = (__bf16)(sum[u][r] * inv);
        ob[u] = __builtin_bit_cast(uint2, x);
    }
    if constexpr (UPW % 2 == 0) {
#pragma unroll
        for (int u = 0; u < UPW; u += 2) {
            // lanes of g = 1 and 3 give their columns of tile u for those that g = 0 and 2 have of tile u + 1: 8 adjacent columns per lane
            const auto x = __builtin_amdgcn_permlane16_swap(ob[u].x, ob[u + 1].x, false, false), y = __builtin_amdgcn_permlane16_swap(ob[u].y, ob[u + 1].y, false, false);
            const u32x4 w = {x[0], y[0], x[1], y[1]};
            if (f < n_rows)
                __builtin_nontemporal_store(w, reinterpret_cast<u32x4_any *>(op + (u + (g & 1)) * 16 + (g >> 1) * 8));
        }
    } else if (f < n_rows) {
#pragma unroll
        for (int u = 0; u < UPW; u++)
            *reinterpret_cast<u32x2_any *>(op + u * 16 + g * 4) = __builtin_bit_cast(u32x2_any, ob[u]);
    }
    if (f >= n_rows)
        return;
    if (ds == 0 && dt0 == 0 && g == 0 && a.lse)
        a.lse[((int64_t)b * a.n_q_heads + head) * a.n_q + row] = lt > 0.0f ? (mt + log2f(lt)) * 0.6931471805599453f : -INFINITY;
}

// keys per tile: 32 where the key groups' tiles fit a workgroup's LDS
template <int D, int NW, int DS>
constexpr int wave_keys() { return D == 64 || (D == 128 && (DS == 4 || NW == 4)) || (D == 256 && DS == 4 && NW == 4) ? 32 : 16; }
template <int D, int NW, int DS, int QT>
using WaveGeom = RowsGeom<D, DS, QT, 1, NW, wave_keys<D, NW, DS>()>;
template <int D, int DS, int QT>
using PairGeom = RowsGeom<D, DS, QT, 2, 4, D == 256 ? 16 : 32>;
template <int D, int DS, int QT>
using QuadGeom = RowsGeom<D, DS, QT, 4, 2, D == 256 ? 16 : 32>;

// one query slot: NW key groups of one wave, QT query tiles and one of DS column slices a workgroup
template <int D, int NW, int DS, int QT, int FORM>
__global__ __launch_bounds__(64 * NW) void attn_wave_kernel(ROWS_PARAMETERS)
{
    attend_rows<D, DS, QT, 1, NW, wave_keys<D, NW, DS>(), FORM>(ROWS_ARGUMENTS);
}

// two query slots: 4 key groups of two waves, 2 * QT query tiles a workgroup
template <int D, int DS, int QT, int FORM>
__global__ __launch_bounds__(512) void attn_pair_kernel(ROWS_PARAMETERS)
{
    attend_rows<D, DS, QT, 2, 4, D == 256 ? 16 : 32, FORM>(ROWS_ARGUMENTS);
}

// four query slots: 2 key groups of four waves, 4 * QT query tiles a workgroup
template <int D, int DS, int QT, int FORM>
__global__ __launch_bounds__(512) void attn_quad_kernel(ROWS_PARAMETERS)
{
    attend_rows<D, DS, QT, 4, 2, D == 256 ? 16 : 32, FORM>(ROWS_ARGUMENTS);
}

// ------------------------------------------------------------------------------------------------
// float32 path: one workgroup of 4 waves per (query row, head, sequence).  D / 4 adjacent lanes share a key, each with four
// dimensions of its K row and of its V row; a wave serves 256 / D keys at a time and each lane U of them per pass, so the score of a
// key is reduced inside its lanes and multiplied with the V row there.  Every wave keeps its own online-softmax state;
// the four meet in LDS at the end.  Latency bound (the tiny configuration reads 0.2 MB): the first pass's K and V rows, the
// query, the parents and the prefix length are all requested before any of them is needed.
// Measured, 4 heads x 8 rows x 104 keys: 19.2 us before (a dependent chain of parent loads, then one V row after the other),
// 4.4 us a call here, the launch and the host included.
// ------------------------------------------------------------------------------------------------
template <int LANES>
__device__ __forceinline__ float sum_lanes(float v)   // over aligned groups of LANES lanes, in every lane of the group
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));   // row_ror:8 of 16 lanes, and so on
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xf, 0xf, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, false));
    if (LANES >= 32)
        v += __shfl_xor(v, 16);
    if (LANES >= 64)
        v += __shfl_xor(v, 32);
    return v;
}

template <int D>
__global__ __launch_bounds__(256) void attn_f32_kernel(AttnArgs a)
{
    constexpr int LPK = D / 4, KPW = 64 / LPK, U = 8, PASS = 4 * KPW * U;   // lanes per key; keys per wave at a time; keys per pass
    __shared__ int32_t s_par[DREAM_MAX_TREE];
    __shared__ __attribute__((aligned(16))) float s_o[4][D];   // (written 16 bytes at a time)
    __shared__ float s_m[4], s_l[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = blockIdx.x, hq = blockIdx.y, b = blockIdx.z;
    const int kvh = hq / a.group;
    const int slot = wave * KPW + lane / LPK, col = lane % LPK;              // this lane's keys: slot + 4 * KPW * u of a pass
    const f32x4 *kb = reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(a.k) + ((int64_t)b * a.n_kv_heads + kvh) * a.s_max * D) + col;
    const f32x4 *vb = reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(a.v) + ((int64_t)b * a.n_kv_heads + kvh) * a.s_max * D) + col;
    f32x4 kr[U], vr[U];
    auto issue = [&](int k0, int64_t rows) {     // keys past `rows` read the last of them; they are masked
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t key = min((int64_t)(k0 + slot + u * 4 * KPW), rows - 1);
            kr[u] = kb[key * LPK];
            vr[u] = vb[key * LPK];
        }
    };
    issue(0, a.s_max);                           // before the prefix length is known: any row of the cache may be read
    const int P0 = a.prefix_len[b];
    const f32x4 q = reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(a.q) + (((int64_t)b * a.n_q + row) * a.n_q_heads + hq) * D)[col];
    int node = row;
    if (a.q_node)
        node = min(max(a.q_node[(int64_t)b * a.n_q + row], 0), a.n_tree - 1);
    if (!a.tree_mask && tid < a.n_tree) {
        const int p = a.parent[(int64_t)b * a.n_tree + tid];
        s_par[tid] = p < tid ? p : -1;           // a walk up the tree always ends
    }
    __syncthreads();
    const NodeMask<4> mask = visible_nodes<4>(a, b, node, s_par);
    const int P = (int)min((int64_t)max(P0, 0), a.s_max - a.n_tree);   // never past the cache, whatever the array holds
    const int kv_len = P + a.n_tree;
    float m_run = -INFINITY, l_run = 0.0f;       // of this wave; l_run of this lane's keys only until the end
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < kv_len; k0 += PASS) {
        if (k0 > 0)
            issue(k0, kv_len);
        float sc[U], mx = -INFINITY;
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int key = k0 + slot + u * 4 * KPW, rel = key - P;
            const bool vis = rel < 0 || (rel < a.n_tree && mask_bit(mask, rel));
            const float dot = sum_lanes<LPK>((q[0] * kr[u][0] + q[1] * kr[u][1]) + (q[2] * kr[u][2] + q[3] * kr[u][3]));
            sc[u] = vis ? dot * a.scale : -INFINITY;
            mx = fmaxf(mx, sc[u]);
        }
        if (KPW >= 4)
            mx = fmaxf(mx, __shfl_xor(mx, 16));
        if (KPW >= 2)
            mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run, mx), m_safe = (m_new == -INFINITY) ? 0.0f : m_new;
        const float alpha = expf(m_run - m_safe);
        l_run *= alpha;
        o *= alpha;
        m_run = m_new;
#pragma unroll
        for (int u = 0; u < U; u++) {
            const float p = expf(sc[u] - m_safe);
            l_run += p;
            if (p != 0.0f)                        // (an invisible key's V row is never used)
                o += vr[u] * p;
        }
    }
    // the lanes that hold other keys of the same dimensions, then the four waves
    if (KPW >= 4) {
        l_run += __shfl_xor(l_run, 16);
#pragma unroll
        for (int i = 0; i < 4; i++)
            o[i] += __shfl_xor(o[i], 16);
    }
    if (KPW >= 2) {
        l_run += __shfl_xor(l_run, 32);
#pragma unroll
        for (int i = 0; i < 4; i++)
            o[i] += __shfl_xor(o[i], 32);
    }
    if (lane < LPK)
        reinterpret_cast<f32x4 *>(s_o[wave])[col] = o;
    if (lane == 0) {
        s_m[wave] = m_run;
        s_l[wave] = l_run;
    }
    __syncthreads();
    if (tid < D) {
        const float m = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3])), ms = (m == -INFINITY) ? 0.0f : m;
        float l = 0.0f, r = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; w++) {
            const float f = expf(s_m[w] - ms);
            l += s_l[w] * f;
            r += s_o[w][tid] * f;
        }
        reinterpret_cast<float *>(a.out)[(((int64_t)b * a.n_q + row) * a.n_q_heads + hq) * D + tid] = l > 0.0f ? r / l : 0.0f;
        if (a.lse && tid == 0)
            a.lse[((int64_t)b * a.n_q_heads + hq) * a.n_q + row] = l > 0.0f ? m + logf(l) : -INFINITY;
    }
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
struct Plan {
    int tiles_per_head, qg, n_qg, n_splits, n_streams, grid, n_groups, kt, pfd;
    int nw;           // waves per workgroup of the shared-tile kernel (4 or 8)
    int mw;           // 64-bit words of a node's visibility mask (1, or 4 for trees above 64 nodes)
    int once;         // 1: the variant whose K/V loads carry the nontemporal hint (one query group per KV head)
    int kg;           // key groups per workgroup of the shared-tile kernel (1; 2 = 8 waves as two groups of 4)
    bool wave_mode;   // attn_wave_kernel, attn_pair_kernel or attn_quad_kernel: waves split the keys of a workgroup, workgroups do not
    int wave_nw;      // waves per workgroup in that mode
    int wave_ds;      // workgroups that share the output columns of a query tile in that mode (1, 2 or 4)
    int wave_qt;      // query tiles per wave in that mode
    int slots;        // query slots of a workgroup in that mode: 1, 2 (attn_pair_kernel) or 4 (attn_quad_kernel)
    int64_t max_kv_len;
    size_t state_floats, off_part, total;
};

// The kernels that cut the work into query tiles and column slices only (attn_wave_kernel, attn_pair_kernel, attn_quad_kernel): one launch, no key split.
// What such a launch costs is what its busiest CU pulls, K and 1 / DS of V per workgroup, as long as all workgroups run at once; so
// the decompositions below are tried from the one that spreads the bytes thinnest, and the first with at most one workgroup per CU is
// taken, while the range is no longer than longest_range() says.  (A workgroup for two tiles where a KV head has one multiplies an empty one: 5 sequences of 32 heads, head_dim 128,
// 10 rows, us with it / without: 5 key tiles 7.4 / 6.1, 20 tiles 11.9 / 11.2, 60 tiles 27.2 / 26.7.)
struct Decomposition {
    int d, slots, ds, qt;
    int tiles_1, tiles_n;    // line against five splits or more with every CU at work, in 32-key tiles, with one query head per KV head and with several (0: not used)
};
const Decomposition DECOMPOSITIONS[] = {
    {128, 1, 4, 1, 52, 72}, {128, 1, 2, 1, 64, 84}, {128, 1, 2, 2, 72, 106}, {128, 1, 2, 3, 60, 76}, {128, 1, 1, 1, 48, 76}, {128, 1, 1, 2, 48, 76}, {128, 2, 1, 2, 0, 76}, {128, 4, 1, 2, 0, 76},
    {64, 1, 2, 1, 90, 108}, {64, 1, 1, 1, 84, 108}, {64, 1, 1, 2, 84, 108}, {64, 2, 1, 2, 84, 0},
    {256, 1, 4, 1, 0, 58}, {256, 1, 4, 2, 0, 60}, {256, 1, 4, 3, 0, 70}, {256, 2, 2, 1, 0, 50}, {256, 2, 2, 2, 0, 52}, {256, 4, 2, 2, 0, 52},
};

// The number of 32-key tiles up to which one launch without key splits beats what the general plan makes of the shape: key splits with a merge launch,
// which cost more to start and less per tile, while few sequences leave CUs idle, or one workgroup for all rows of a KV head.  `line`: where the two meet
// against five splits or more with every CU at work; earlier when fewer CUs pull, later against fewer splits.  Against two or none the single
// launch is ahead at every length measured, up to 128 tiles.
// The lines are those of least regret over 16 groupings of heads, 1 to 32 sequences, 8 to 64 rows and 7 to 104 tiles, the caches of 24 to 48 layers in turn:
// against three splits or more the rule takes 0.2 % more than the better of both on average (one line per decomposition, whatever it replaces: 0.7 %).  The worst
// are single sequences whose caches of all layers fit the memory-side cache, where the single launch is ahead for longer (8 heads, 64 rows, 48 tiles 9.2 / 12.6).  us, single launch /
// general plan, last length below the line and first above:
//   head_dim 128: 32 heads, 1 sequence, 8 rows, 128 workgroups, 40 tiles 12.0 / 12.1, 44 tiles 12.6 / 12.5; 2 sequences, against four splits, 60 tiles
//   17.4 / 18.0, 64 tiles 19.4 / 19.5; 33 rows in 2 slices, 56 tiles 15.2 / 15.6, 60 tiles 16.1 / 15.7; 64 rows 64 tiles 17.5 / 17.7, 70 tiles 17.8 / 17.9; 8 KV heads, groups
//   of 4, 64 rows, 78 tiles 17.8 / 18.2, 90 tiles 19.9 / 19.3; against two splits, 4 sequences of 8 rows, 104 tiles 38.0 / 41.0
//   head_dim 64: 32 heads, 1 sequence, 8 rows, 64 workgroups, 60 tiles 10.4 / 10.7, 64 tiles 11.4 / 10.7; 64 rows, 256 workgroups, 90 tiles 13.5 / 13.9, 104 tiles
//   15.1 / 14.8; 3 sequences of 8 rows, against two splits, 104 tiles 19.8 / 22.6
//   head_dim 256, 8 KV heads, groups of 2: 64 rows 56 tiles 20.2 / 21.7, 64 tiles 22.5 / 21.4; 2 sequences of 8 rows, 64 workgroups, 36 tiles 16.0 / 16.1, 44 tiles 18.5 / 17.1
// While the memory-side cache holds the caches (`near`), every workgroup pulls faster and few of them are no reason to change early (but for groups of 3 heads of 256, whose rows fill
// few slices: 3 sequences of 8 KV heads, 44 tiles equal, 63 tiles 25.5 / 22.2): at most 8 % behind at the last length
// over 16 groupings, 1 to 8 sequences, 1 to 60 rows and 28 to 160 tiles, where the lines above lost up to 1.5x.  us, single launch / general plan, cross-attention of 10 rows: head_dim 128, 32 heads,
// 1 sequence 64 tiles 10.8 / 13.2, 90 tiles 15.2 / 15.2, 100 tiles 16.3 / 15.6; 8 KV heads, groups of 2, 3 sequences 100 tiles 15.9 / 15.9, 112 tiles 17.6 / 16.7, groups of 4, 4 sequences 80 tiles
// 14.6 / 18.2, 126 tiles 19.9 / 21.3; head_dim 64, 32 heads, 1 sequence 64 tiles 8.2 / 9.9, 112 tiles 11.7 / 11.9, 126 tiles 12.9 / 12.3; against two splits, 3 sequences, 126 tiles 17.2 / 25.4;
// head_dim 256, groups of 2, 2 sequences 64 tiles 18.4 / 19.5, 72 tiles 20.1 / 20.2, 80 tiles 21.6 / 21.2.  Verification of one sequence: 8 heads of 128, 60 rows, 64 tiles 11.0 / 13.5.
int64_t longest_range(const dream_attn_desc *d, int n_qtiles, int64_t workgroups, int slots, int line, bool near)
{
    const int G = d->n_q_heads / d->n_kv_heads;
    const int64_t splits = 256 / ((int64_t)d->batch * d->n_kv_heads * ceil_div(n_qtiles, 4));
    if (splits < 3)
        return d->head_dim == 256 ? (G == 1 ? 96 : 128) : near || (slots > 1 && G > 1) ? 1 << 30 : G == 1 ? 120 : 160;
    const int64_t cold = line * (384 + workgroups) / 640;
    const int64_t tiles = !near ? cold : d->head_dim == 64 ? std::max(line * 5 / 4, 112) : d->head_dim == 128 ? std::max(line * 5 / 4, G == 1 ? 90 : 100) : G == 3 ? std::max<int64_t>(cold, 45) : std::max(line * 5 / 4, 72);
    return splits == 4 ? tiles * 6 / 5 : splits == 3 ? tiles * 8 / 5 : tiles;
}

bool make_wave_plan(const dream_attn_desc *d, int n_q, int64_t max_kv_len, bool near, Plan *p)
{
    const int G = d->n_q_heads / d->n_kv_heads;
    const int64_t base = (int64_t)d->batch * d->n_kv_heads;
    const int64_t places = (base + 7) / 8 * 8;       // 8 times the KV heads of the XCD that has most: one workgroup per CU counts these
    const int tiles = ceil_div(max_kv_len, 32), rows = ceil_div((int64_t)G * n_q, 16);
    const int n_qtiles = G * ceil_div(n_q, 16);      // as many as the heads' rows would need one head after the other
    p->wave_mode = false;
    p->slots = 1;
    if (d->dtype != DREAM_BF16 || q_tiles_override() != 0 || kv_splits_override() != 0 || tile_waves_override() != 0 || n_qtiles > 16 || G > 4 ||
        base * n_qtiles < 32 || d->s_max * d->head_dim >= (1ll << 30))
        return false;
    if (G == 3 || (G == 1 && d->head_dim == 256)) {
        // one query tile a workgroup in as many column slices as leave one workgroup per CU, or two tiles
        if (places * n_qtiles > (d->head_dim <= 128 ? 512 : 256))
            return false;
        p->wave_ds = 1;
        while (p->wave_ds < 4 && places * n_qtiles * p->wave_ds * 2 <= 256 && d->head_dim / (p->wave_ds * 2) >= 32)
            p->wave_ds *= 2;
        p->wave_qt = places * n_qtiles > 256 ? 2 : 1;
        // (3 tiles a head are two workgroups: 20 sequences of 8 KV heads, head_dim 128, 64 key tiles: 320 workgroups 48 us, the 160 of the plan without 32)
        const int64_t workgroups = base * ceil_div(rows, p->wave_qt) * p->wave_ds;
        if (places * ceil_div(rows, p->wave_qt) * p->wave_ds > 256)
            return false;
        // us on both sides of a line, 8 KV heads in groups of 3: head_dim 64, 2 sequences, 96 tiles 14.9 / 15.6, 128 tiles 19.2 / 17.5; head_dim 128, unsliced, 48 tiles 15.6 / 17.1,
        // 64 tiles 19.7 / 19.9; head_dim 256, 26 tiles 18.2 / 22.2, 40 tiles 26.8 / 25.5; one head of 256, 2 slices, 48 tiles 23.2 / 24.4, 56 tiles 26.3 / 25.2
        static const int LINES[3][3] = {{108, 108, 108}, {64, 74, 76}, {36, 50, 54}};    // by head_dim; unsliced, 2 slices, 4
        if (tiles > longest_range(d, n_qtiles, workgroups, 1, LINES[d->head_dim / 128][p->wave_ds / 2], near))
            return false;
    } else {
        const Decomposition *use = nullptr;
        for (const Decomposition &c : DECOMPOSITIONS)
            if (!use && c.d == d->head_dim && places * ceil_div(rows, c.slots * c.qt) * c.ds <= 256)
                use = &c;
        const int line = !use ? 0 : G == 1 ? use->tiles_1 : use->tiles_n;
        if (!line)
            return false;
        const int units = ceil_div(rows, use->slots * use->qt);
        if (tiles > longest_range(d, n_qtiles, base * units * use->ds, use->slots, line, near))
            return false;
        // Three exceptions.  Four slots for all rows of a KV head start slower than the 8 waves of the shared-tile kernel, which do the same, the more so
        // the more CUs are at work: 18 sequences of 17 rows 18 tiles 17.9 / 18.0, 24 sequences
        // 8 tiles 13.2 / 11.5 us, 16 tiles 17.9 / 17.1, 24 tiles 22.2 / 22.2, 32 tiles 26.7 / 28.0, 32 sequences 30 tiles 28.4 / 28.5.  Up to 96 KV heads with 4 tiles each, and pairs of heads of 64,
        // change earlier than they would have to (3 sequences, 64 rows, 52 tiles 22.3 / 26.4, 64 tiles 25.8 / 30.2; 5 sequences, 64 rows, 40 tiles 14.5 / 15.1, 52 tiles 17.4 / 17.6, 8
        // sequences 52 tiles 20.7 / 23.5).
        if (use->slots == 4 && use->d == 128 && units == 1 && tiles < 8 + base / 12)
            return false;
        if (G == 1 && use->ds == 1 && use->qt == 2 && (use->d == 128 ? base <= 96 && tiles > 48 : use->slots == 2 && tiles > 40))
            return false;
        p->slots = use->slots;
        p->wave_ds = use->ds;
        p->wave_qt = use->qt;
    }
    p->wave_mode = true;
    // 4 waves while each has about one tile (5 tiles: 6.8 us with 4, 6.9 with 8), and at head_dim 256 with one query tile, where a wave's 32
    // keys of 4 waves and 16 keys of 8 take the same LDS (42 tiles: 16.4 us with 4, 15.9 with 8)
    p->wave_nw = 8;
    if (p->slots == 1 && (d->head_dim == 256 ? p->wave_qt == 1 : p->wave_ds == 1 && tiles <= 5))
        p->wave_nw = 4;
    p->qg = 1;
    // The grid has a workgroup for every tile that the heads would need one after the other while each has a CU of its own: those beyond the rows
    // end at once and cost nothing there (60 rows of 4 heads, 8 KV heads, 1340 keys: 256 workgroups 9.65 us, the 240 with rows 9.6).  With more of
    // them than CUs, two that work would share one while others idle (3 sequences of 17 rows, 384 workgroups and 240: 23.7 / 12.6 us at 1417 keys, 35.5 / 18.5 at 2417).
    p->n_qg = p->wave_qt == 1 && p->slots == 1 && places * n_qtiles * p->wave_ds <= 256 ? n_qtiles : rows;
    p->n_splits = 1;
    p->n_groups = p->n_streams = (int)base;
    p->grid = 0;
    p->kt = p->pfd = 1;
    p->state_floats = 0;
    p->off_part = DREAM_WORKSPACE_MIN_BYTES;
    p->total = DREAM_WORKSPACE_MIN_BYTES;
    p->max_kv_len = max_kv_len;
    return true;
}

// direct: q and the caches are 16-byte aligned, as loads straight to LDS need them.  near: the memory-side cache still holds the caches
int make_plan(const dream_attn_desc *d, int n_q, int64_t max_kv_len, bool direct, bool near, Plan *p)
{
    const int G = d->n_q_heads / d->n_kv_heads;
    if (make_wave_plan(d, n_q, max_kv_len, near, p)) {
        if (direct)
            return 0;
        p->wave_mode = false;
        p->slots = 1;
    } else {
        direct = true;
    }
    p->wave_nw = p->wave_ds = 0;
    p->wave_qt = 1;
    p->tiles_per_head = ceil_div(n_q, 16);
    const int n_qtiles = G * p->tiles_per_head;
    const int qg_max = d->head_dim == 256 ? 2 : 4;   // accumulator registers bound the query tiles per wave
    const int64_t base = (int64_t)d->batch * d->n_kv_heads;
    const int tiles = ceil_div(max_kv_len, 32);
    // throughput regime: as many query tiles per wave as registers allow, so that a K/V byte read from
    // LDS serves the most rows.  Latency regime (too few streams to fill the chip): one tile per wave keeps
    // the per-workgroup state small; the query groups of a KV head then re-read its K/V through L2.
    int qg = q_tiles_override();
    if (qg <= 0) {
        qg = n_qtiles <= 4 ? 1 : n_qtiles <= 8 ? 2 : 4;
        if (qg > qg_max)
            qg = qg_max;
        if (base * ceil_div(n_qtiles, 4 * qg) < 256)
            qg = 1;
        // measured at 32 sequences of a 4-way grouped-query model: below about four workgroups per CU the
        // chip hides latency better with more, smaller workgroups than it gains from sharing LDS reads
        // (head_dim 256 is the exception: its tiles are twice the bytes to re-read)
        while (d->head_dim <= 128 && qg > 1 && base * ceil_div(n_qtiles, 4 * qg) < 1024)
            qg /= 2;
    }
    if (qg > qg_max)
        qg = qg_max;
    if (qg != 1 && qg != 2 && qg != 4)
        qg = 1;
    p->qg = qg;
    p->nw = 4;
    p->mw = 1;
    p->once = 0;
    p->kg = 1;
    p->n_qg = ceil_div(n_qtiles, 4 * qg);
    // grouped-query shapes with more 4-wave workgroups than the chip runs well: 8 waves share one LDS tile, so the 8-16
    // query tiles of a KV head are served by ONE workgroup (K/V leave L2 once per head instead of once per 4 query tiles)
    // while the CU still holds 8 waves.  head_dim 64 tiles are too small to spread over 512 threads; with more than 16
    // (8 at head_dim 256) query tiles a KV head takes several workgroups.  The lines, from 42 key tiles at 4-32 sequences:
    // head_dim 128, 16 query tiles: 47-52 us whatever the number of workgroups up to one per CU, against 38-42 us of two 4-wave
    // workgroups per CU and 62-76 us of more; up to 8 query tiles: 33-36 us against 37-40 us of two per CU; head_dim 256: 58-70 us
    // against 52 us of one per CU and 102 us of two, and with up to 4 query tiles (where it replaces a second
    // key split as well, unless the range is long) 41-50 us against 50 us of one per CU and 37-43 us of two splits (32 key
    // tiles: 34 us against 35-38; three splits win earlier, 72 workgroups: 27.1 against 27.8 us at 24 tiles, 33.6 against 30.7 at 32).
    // The other lines hold at every length from 8 to 130 tiles: 17 sequences, head_dim 128, 16 query tiles 16.6 against 20.2 and 125
    // against 174 us, 8 query tiles 12.1 against 13.3 and 94 against 105 us, head_dim 256 18.3 against 31.2 and 162 against 283 us,
    // its 4 query tiles 14.4 against 16.6 and 117 against 142 us; 16 sequences are still faster with 4 waves (114.6 against 130.2,
    // 62.9 against 98.6, 147 against 164 us at 130 tiles).
    {
        const int tw = tile_waves_override();
        const int qg8_max = d->head_dim == 256 ? 1 : 2;
        int qg8 = q_tiles_override() > 0 ? (q_tiles_override() > qg8_max ? qg8_max : q_tiles_override()) : (n_qtiles > 8 ? qg8_max : 1);
        const bool can8 = d->dtype == DREAM_BF16 && d->head_dim >= 128 && kv_splits_override() <= 1 && tw != 4;
        const int64_t wg4 = base * ceil_div(n_qtiles, 4);
        const bool few = n_qtiles <= 4;        // (at head_dim 128: see the two key groups below)
        const bool full = few ? d->head_dim == 256 && (wg4 > 128 || (wg4 > 64 && tiles <= (wg4 <= 85 ? 24 : 32))) : wg4 > (qg8 == 2 ? 512 : 256);
        const bool want8 = (tw == 8 && !few) || (tw == 0 && q_tiles_override() == 0 && full);
        // (the 8-wave variants read K/V with the nontemporal hint, so a KV head must not need two of them)
        if (can8 && want8 && ceil_div(n_qtiles, 8 * qg8) == 1) {
            p->nw = 8;
            p->qg = qg = qg8;
            p->n_qg = 1;
            p->once = 1;
        }
    }
    int s = kv_splits_override();
    if (p->nw == 8 || !direct)     // (a call in place of one without splits has a workspace for none)
        s = 1;
    if (s <= 0) {
        // at most one workgroup per CU: a few more leave most of the chip waiting for the last ones (96 groups of head_dim 256,
        // 42 key tiles: 49.8 us in 3 splits, 37.4 us in 2; 160 groups: 65.7 us in 2, 52.1 us in 1)
        s = (int)(256 / (base * p->n_qg));
        if (s > 8)
            s = 8;                           // more splits cost more in the merge than they save
        // ... as do two or three of a short range whose workgroups can have two key groups instead.  Unsplit against split, us at
        // head_dim 128 (64 crosses at the same lengths): three splits, 72 groups: 15.9 / 17.2 at 24 key tiles, 18.9 / 18.4 at 32,
        // 30.9 / 24.8 at 64, 84 groups: 18.9 / 20.5 at 32, 26.5 / 25.4 at 52; two splits, 88 groups: 22.6 / 23.3 at 42, 26.4 / 26.3
        // at 52, 31.1 / 29.6 at 64, 128 groups: 16.4 / 20.7 at 24, 31.3 / 32.3 at 64, 37.8 / 36.5 at 80
        const int64_t groups = base * p->n_qg;
        if (d->head_dim <= 128 && s <= 3 && tiles <= (s == 3 ? 32 : groups <= 96 ? 52 : 64))
            s = 1;
    }
    if (s > tiles)
        s = tiles;
    if (s < 1)
        s = 1;
    const int64_t groups = base * p->n_qg;
    if (groups * qg * p->nw > 0x7fffffff)
        s = 1;
    p->n_splits = s;
    p->n_groups = (int)groups;
    p->n_streams = (int)(base * s);
    p->grid = ceil_div(p->n_streams, 8) * 8 * p->n_qg;
    // short streams (latency regime): the whole share of a workgroup is one step, everything in flight at once;
    // long streams: one tile per step (two at head_dim 64, whose tiles are half the bytes), two steps in flight
    const int tps = ceil_div(tiles, s);
    if (qg == 1 && d->head_dim <= 128 && tps <= 4) {
        p->kt = tps < 2 ? 2 : tps;
        p->pfd = 1;
    } else {
        p->kt = (qg == 1 && d->head_dim == 64) ? 2 : 1;
        p->pfd = 2;
        // the widest variants keep one step in flight: with two their accumulators and staging registers no
        // longer fit the 512 registers of a wave (same speed, no spills)
        if ((qg == 4 && d->head_dim == 128) || (qg == 2 && d->head_dim == 256))
            p->pfd = 1;
    }
    if (p->nw == 8) {
        p->kt = 1;
        p->pfd = DREAM_W8_PFD;
    } else if (qg == 1 && p->pfd == 2) {
        p->once = p->n_qg == 1;
        // shapes that leave a CU with at most DREAM_KG2_MAX_WG 4-wave workgroups: 8 waves as two key groups (several query
        // groups per KV head, 42 key tiles, 256 workgroups: 29.8 us with 4 waves, 23.8 us)
        const int tw = tile_waves_override();
        if (s == 1 && d->head_dim <= 128 && tw != 4 && (tw == 8 || (groups <= 256 * DREAM_KG2_MAX_WG && (p->n_qg == 1 || q_tiles_override() == 0)))) {
            p->nw = 8;
            p->kg = 2;
        }
    }
    p->state_floats = (size_t)qg * (d->head_dim / 16) * 256 + (size_t)qg * 2 * 64;
    p->off_part = DREAM_WORKSPACE_MIN_BYTES;
    p->total = p->off_part + (s > 1 ? (size_t)groups * s * 4 * p->state_floats * sizeof(float) : 0);
    if (d->dtype == DREAM_F32)
        p->total = DREAM_WORKSPACE_MIN_BYTES;
    return 0;
}

// Trees above 64 nodes: the shared-tile kernel with four mask words, one query tile per wave, the key range unsplit
// (no split states, so the workspace need never exceeds what the query for any other shape returns), streamed.
void make_wide_plan(const dream_attn_desc *d, int n_q, Plan *p)
{
    const int G = d->n_q_heads / d->n_kv_heads;
    const int64_t base = (int64_t)d->batch * d->n_kv_heads;
    p->tiles_per_head = ceil_div(n_q, 16);
    p->wave_mode = false;
    p->wave_nw = p->wave_ds = p->wave_qt = 0;
    p->slots = 1;
    p->qg = 1;
    p->nw = 4;
    p->mw = 4;
    p->once = 0;
    p->kg = 1;
    p->n_qg = ceil_div(G * p->tiles_per_head, 4);
    p->n_splits = 1;
    p->n_groups = (int)(base * p->n_qg);
    p->n_streams = (int)base;
    p->grid = ceil_div(p->n_streams, 8) * 8 * p->n_qg;
    p->kt = d->head_dim == 64 ? 2 : 1;
    p->pfd = 2;
    p->state_floats = 0;
    p->off_part = DREAM_WORKSPACE_MIN_BYTES;
    p->total = DREAM_WORKSPACE_MIN_BYTES;
}

int validate_desc(const dream_attn_desc *d, const char *who)
{
    if (!d)
        return fail(DREAM_ERR_INVALID_ARG, "%s: desc is NULL", who);
    if (d->batch < 1 || d->n_q_heads < 1 || d->n_kv_heads < 1 || d->s_max < 1)
        return fail(DREAM_ERR_INVALID_ARG, "%s: batch, head counts and s_max must be positive", who);
    if (d->n_q_heads % d->n_kv_heads)
        return fail(DREAM_ERR_INVALID_ARG, "%s: n_q_heads %d is not a multiple of n_kv_heads %d", who, d->n_q_heads, d->n_kv_heads);
    if (d->head_dim != 64 && d->head_dim != 128 && d->head_dim != 256)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: head_dim %d not in {64,128,256}", who, d->head_dim);
    if (d->dtype != DREAM_F32 && d->dtype != DREAM_BF16)
        return fail(DREAM_ERR_INVALID_ARG, "%s: unknown dtype %d", who, d->dtype);
    if (d->batch > 65535 || d->n_q_heads > 65535)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: batch and n_q_heads are limited to 65535", who);
    return DREAM_OK;
}

template <int D, int QG, int KT, int PFD, int NW = 4, int MW = 1, bool ONCE = false, int KG = 1>
int ensure_bf16_lds()
{
    static std::atomic<uint64_t> done{0};
    return raise_lds_limit(done, reinterpret_cast<const void *>(&attn_bf16_kernel<D, QG, KT, PFD, NW, MW, ONCE, KG>), Geom<D, QG, KT * KG>::LDS_BYTES, "attention");
}

template <int D, int QG, int KT, int PFD, int NW = 4, int MW = 1, bool ONCE = false, int KG = 1>
int launch_bf16(const AttnArgs &a, const Plan &p, hipStream_t st)
{
    using G = Geom<D, QG, KT * KG>;
    if (int rc = ensure_bf16_lds<D, QG, KT, PFD, NW, MW, ONCE, KG>())
        return rc;
    if (ONCE && a.n_qg != 1)
        return fail(DREAM_ERR_INVALID_ARG, "attention: the read-once kernel variant needs one query group per KV head, not %d", a.n_qg);
    if (NW != 4 && p.n_splits != 1)
        return fail(DREAM_ERR_INVALID_ARG, "attention: the 8-wave shared-tile kernel does not split the key range");
    if (a.mask_words > MW)
        return fail(DREAM_ERR_INVALID_ARG, "attention: a tree of %d nodes needs %d mask words, this kernel has %d", a.n_tree, a.mask_words, MW);
    hipLaunchKernelGGL((attn_bf16_kernel<D, QG, KT, PFD, NW, MW, ONCE, KG>), dim3(p.grid), dim3(64 * NW), G::LDS_BYTES, st, a);
    int rc = check_launch("attn_bf16_kernel");
    if (rc || p.n_splits == 1)
        return rc;
    hipLaunchKernelGGL((attn_merge_kernel<D, QG>), dim3(p.n_groups * 4 * QG), dim3(256), 0, st, a);
    return check_launch("attn_merge_kernel");
}

template <class G>
constexpr bool has_hint(int slices) { return slices != 4 && !G::SWAPPED; }

template <int D, int NW, int DS, int QT>
int ensure_wave_lds()
{
    using G = WaveGeom<D, NW, DS, QT>;
    constexpr int hinted = has_hint<G>(DS) ? READ_ONCE : READ_PLAIN, turned = G::TURNED ? READ_TURNED : READ_PLAIN, brief = G::SWAPPED ? READ_PLAIN : READ_SHORT;     // (the plain form again where there is no such form)
    static std::atomic<uint64_t> done[4];
    int rc = raise_lds_limit(done[0], reinterpret_cast<const void *>(&attn_wave_kernel<D, NW, DS, QT, READ_PLAIN>), G::BYTES, "attention");
    rc = rc ? rc : raise_lds_limit(done[1], reinterpret_cast<const void *>(&attn_wave_kernel<D, NW, DS, QT, hinted>), G::BYTES, "attention");
    rc = rc ? rc : raise_lds_limit(done[2], reinterpret_cast<const void *>(&attn_wave_kernel<D, NW, DS, QT, turned>), G::BYTES, "attention");
    return rc ? rc : raise_lds_limit(done[3], reinterpret_cast<const void *>(&attn_wave_kernel<D, NW, DS, QT, brief>), G::BYTES, "attention");
}

#define ROWS_OF(a) a.prefix_len, a.q, a.k, a.tree_mask ? nullptr : a.parent, (uint32_t)a.n_kv_heads | (uint32_t)a.group << 16, (uint32_t)a.n_q | (uint32_t)a.n_tree << 16, a.spread, a.nq_magic, (uint32_t)a.s_max, (uint32_t)a.n_streams, a

// With few keys most waves of the first step have none, and would pull rows that nobody needs: from three quarters of a step on they are asked for before it is known how many there are.
// us a launch, asked for behind the prefix length / ahead of it, steps of 256 keys: 2 sequences of 16 heads of 128, 18 rows, 104 keys 4.17 / 4.44, 170 keys 4.41 / 4.54, 200 keys 4.54 / 4.56, 240 keys 4.58 / 4.49,
// 3 sequences of 32 heads of 64, 17 rows, 170 keys 4.73 / 4.66, 200 keys 4.95 / 4.69; steps of 128: 4 sequences of 32 heads of 128, 60 rows, 64 keys 6.06 / 6.44, 96 keys 6.64 / 6.78, 104 keys 6.70 / 6.64,
// 120 keys 7.02 / 6.88; 33 rows 64 keys 5.59 / 5.94, 120 keys 6.37 / 6.53, 190 keys 7.13 / 6.88.
// (A sequence of fewer keys beside longer ones, or under a max_kv_len far above its length, still pays: 3 of 54 keys, 39 rows of 32 on 8 heads of 128, max_kv_len 1500, 5.01 / 5.23; at worst
// 4 of 66 keys, 10 rows of 16 heads of 128, 4.55 / 4.95; from 300 keys on the keys asked for early gain.)
template <class G>
bool short_range(const Plan &p) { return p.max_kv_len * 4 < G::STEP_KEYS * 3; }

// `per_head` workgroups for every KV head of every sequence, as attend_rows reads them
dim3 stream_grid(const AttnArgs &a, int per_head)
{
    return a.spread ? dim3(8 * per_head, ceil_div(a.n_streams, 8)) : dim3(8 * per_head, a.n_kv_heads / 8, a.n_streams / a.n_kv_heads);
}

template <int D, int NW, int DS, int QT>
int launch_wave(const AttnArgs &a, const Plan &p, hipStream_t st)
{
    if (int rc = ensure_wave_lds<D, NW, DS, QT>())
        return rc;
    using G = WaveGeom<D, NW, DS, QT>;
    const dim3 grid = stream_grid(a, ceil_div(a.n_qg, QT) * DS);
    auto *kernel = &attn_wave_kernel<D, NW, DS, QT, READ_PLAIN>;
    if constexpr (has_hint<G>(DS))
        kernel = a.once ? &attn_wave_kernel<D, NW, DS, QT, READ_ONCE> : kernel;
    if constexpr (G::TURNED)
        kernel = a.turn ? &attn_wave_kernel<D, NW, DS, QT, READ_TURNED> : kernel;
    if constexpr (!G::SWAPPED)
        kernel = short_range<G>(p) ? &attn_wave_kernel<D, NW, DS, QT, READ_SHORT> : kernel;
    hipLaunchKernelGGL(kernel, grid, dim3(64 * NW), G::BYTES, st, ROWS_OF(a));
    return check_launch("attn_wave_kernel");
}

template <int D, int DS, int QT>
int ensure_pair_lds()
{
    using G = PairGeom<D, DS, QT>;
    static std::atomic<uint64_t> done[3];
    int rc = raise_lds_limit(done[0], reinterpret_cast<const void *>(&attn_pair_kernel<D, DS, QT, READ_PLAIN>), G::BYTES, "attention");
    rc = rc ? rc : raise_lds_limit(done[1], reinterpret_cast<const void *>(&attn_pair_kernel<D, DS, QT, READ_ONCE>), G::BYTES, "attention");
    return rc ? rc : raise_lds_limit(done[2], reinterpret_cast<const void *>(&attn_pair_kernel<D, DS, QT, READ_SHORT>), G::BYTES, "attention");
}

template <int D, int DS, int QT>
int launch_pair(const AttnArgs &a, const Plan &p, hipStream_t st)
{
    if (int rc = ensure_pair_lds<D, DS, QT>())
        return rc;
    using G = PairGeom<D, DS, QT>;
    const dim3 grid = stream_grid(a, ceil_div(a.n_qg, 2 * QT) * DS);
    auto *kernel = short_range<G>(p) ? &attn_pair_kernel<D, DS, QT, READ_SHORT> : a.once ? &attn_pair_kernel<D, DS, QT, READ_ONCE> : &attn_pair_kernel<D, DS, QT, READ_PLAIN>;
    hipLaunchKernelGGL(kernel, grid, dim3(512), G::BYTES, st, ROWS_OF(a));
    return check_launch("attn_pair_kernel");
}

template <int D, int DS, int QT>
int ensure_quad_lds()
{
    using G = QuadGeom<D, DS, QT>;
    static std::atomic<uint64_t> done[3];
    int rc = raise_lds_limit(done[0], reinterpret_cast<const void *>(&attn_quad_kernel<D, DS, QT, READ_PLAIN>), G::BYTES, "attention");
    rc = rc ? rc : raise_lds_limit(done[1], reinterpret_cast<const void *>(&attn_quad_kernel<D, DS, QT, READ_ONCE>), G::BYTES, "attention");
    return rc ? rc : raise_lds_limit(done[2], reinterpret_cast<const void *>(&attn_quad_kernel<D, DS, QT, READ_SHORT>), G::BYTES, "attention");
}

template <int D, int DS, int QT>
int launch_quad(const AttnArgs &a, const Plan &p, hipStream_t st)
{
    if (int rc = ensure_quad_lds<D, DS, QT>())
        return rc;
    using G = QuadGeom<D, DS, QT>;
    const dim3 grid = stream_grid(a, ceil_div(a.n_qg, 4 * QT) * DS);
    auto *kernel = short_range<G>(p) ? &attn_quad_kernel<D, DS, QT, READ_SHORT> : a.once ? &attn_quad_kernel<D, DS, QT, READ_ONCE> : &attn_quad_kernel<D, DS, QT, READ_PLAIN>;
    hipLaunchKernelGGL(kernel, grid, dim3(512), G::BYTES, st, ROWS_OF(a));
    return check_launch("attn_quad_kernel");
}

// Every bf16 kernel variant the launch plan can choose, in one table: the plan names a variant by
// (kernel family, head_dim, three template arguments); the table gives its launcher and the routine that raises
// its dynamic-LDS limit.  The launch, dream_init, dream_attn_plan_describe and dream_attn_variants all read it.
enum { FAMILY_TILE = 0, FAMILY_WAVE = 1, FAMILY_PAIR = 2, FAMILY_QUAD = 4 };
struct Variant {
    int family, d, p1, p2, p3, p4, p5, p6, p7;   // tile: (QG, KT, PFD, waves, mask words, read-once, key groups); wave: (NW, DS, QT, 0, 1, 0, 1)
    int (*launch)(const AttnArgs &, const Plan &, hipStream_t);
    int (*ensure)();
};
#define TILE_VARIANT(D, QG, KT, PFD) {FAMILY_TILE, D, QG, KT, PFD, 4, 1, 0, 1, &launch_bf16<D, QG, KT, PFD>, &ensure_bf16_lds<D, QG, KT, PFD>}
#define ONCE_VARIANT(D, QG, KT, PFD) {FAMILY_TILE, D, QG, KT, PFD, 4, 1, 1, 1, &launch_bf16<D, QG, KT, PFD, 4, 1, true>, &ensure_bf16_lds<D, QG, KT, PFD, 4, 1, true>}
#define KG2_VARIANT(D, QG, KT, PFD) {FAMILY_TILE, D, QG, KT, PFD, 8, 1, 1, 2, &launch_bf16<D, QG, KT, PFD, 8, 1, true, 2>, &ensure_bf16_lds<D, QG, KT, PFD, 8, 1, true, 2>}
#define KG2S_VARIANT(D, QG, KT, PFD) {FAMILY_TILE, D, QG, KT, PFD, 8, 1, 0, 2, &launch_bf16<D, QG, KT, PFD, 8, 1, false, 2>, &ensure_bf16_lds<D, QG, KT, PFD, 8, 1, false, 2>}
#define WIDE_VARIANT(D, QG, KT, PFD) {FAMILY_TILE, D, QG, KT, PFD, 4, 4, 0, 1, &launch_bf16<D, QG, KT, PFD, 4, 4>, &ensure_bf16_lds<D, QG, KT, PFD, 4, 4>}
#define TILE8_VARIANT(D, QG, KT, PFD) {FAMILY_TILE, D, QG, KT, PFD, 8, 1, 1, 1, &launch_bf16<D, QG, KT, PFD, 8, 1, true>, &ensure_bf16_lds<D, QG, KT, PFD, 8, 1, true>}
#define WAVE_VARIANT(D, NW, DS, QT) {FAMILY_WAVE, D, NW, DS, QT, 0, 1, 0, 1, &launch_wave<D, NW, DS, QT>, &ensure_wave_lds<D, NW, DS, QT>}
#define PAIR_VARIANT(D, DS, QT) {FAMILY_PAIR, D, 8, DS, QT, 0, 1, 0, 1, &launch_pair<D, DS, QT>, &ensure_pair_lds<D, DS, QT>}
#define QUAD_VARIANT(D, DS, QT) {FAMILY_QUAD, D, 8, DS, QT, 0, 1, 0, 1, &launch_quad<D, DS, QT>, &ensure_quad_lds<D, DS, QT>}
const Variant VARIANTS[] = {
    // shared-tile kernel, one query tile per wave: a short key range in one step (2-4 tiles), or streamed
    TILE_VARIANT(64, 1, 2, 1), TILE_VARIANT(64, 1, 3, 1), TILE_VARIANT(64, 1, 4, 1), TILE_VARIANT(64, 1, 2, 2),
    TILE_VARIANT(128, 1, 2, 1), TILE_VARIANT(128, 1, 3, 1), TILE_VARIANT(128, 1, 4, 1), TILE_VARIANT(128, 1, 1, 2),
    TILE_VARIANT(256, 1, 1, 2),
    // several query tiles per wave
    TILE_VARIANT(64, 2, 1, 2), TILE_VARIANT(64, 4, 1, 2), TILE_VARIANT(128, 2, 1, 2), TILE_VARIANT(128, 4, 1, 1), TILE_VARIANT(256, 2, 1, 1),
    // streamed, the workgroup the only reader of its K/V rows (one query group per KV head): name arguments ...,4,1,1
    ONCE_VARIANT(64, 1, 2, 2), ONCE_VARIANT(128, 1, 1, 2), ONCE_VARIANT(256, 1, 1, 2),
    // the same with 8 waves as two key groups (few streams per CU): name arguments ...,8,1,1,2
    KG2_VARIANT(64, 1, 2, 2), KG2_VARIANT(128, 1, 1, 2),
    // ... and with several query groups per KV head: name arguments ...,8,1,0,2
    KG2S_VARIANT(64, 1, 2, 2), KG2S_VARIANT(128, 1, 1, 2),
    // 8 waves per workgroup (unsplit key range, grouped queries, always the only reader): a fifth name argument 8
    TILE8_VARIANT(128, 1, 1, DREAM_W8_PFD), TILE8_VARIANT(128, 2, 1, DREAM_W8_PFD), TILE8_VARIANT(256, 1, 1, DREAM_W8_PFD),
    // trees of 65-256 nodes (four mask words): a sixth name argument 4
    WIDE_VARIANT(64, 1, 2, 2), WIDE_VARIANT(128, 1, 1, 2), WIDE_VARIANT(256, 1, 1, 2),
    // one query slot: (waves, column slices, query tiles per workgroup)
    WAVE_VARIANT(64, 8, 1, 1), WAVE_VARIANT(64, 8, 2, 1), WAVE_VARIANT(64, 4, 1, 1),
    WAVE_VARIANT(64, 8, 1, 2), WAVE_VARIANT(64, 4, 1, 2),
    WAVE_VARIANT(128, 8, 1, 1), WAVE_VARIANT(128, 8, 2, 1), WAVE_VARIANT(128, 8, 4, 1), WAVE_VARIANT(128, 4, 1, 1),
    WAVE_VARIANT(128, 8, 1, 2), WAVE_VARIANT(128, 4, 1, 2),
    WAVE_VARIANT(256, 4, 1, 1), WAVE_VARIANT(256, 4, 2, 1), WAVE_VARIANT(256, 4, 4, 1),
    WAVE_VARIANT(128, 8, 2, 2), WAVE_VARIANT(128, 8, 2, 3), WAVE_VARIANT(256, 8, 4, 2), WAVE_VARIANT(256, 8, 4, 3),
    // two query slots: (column slices, query tiles per slot)
    PAIR_VARIANT(64, 1, 2), PAIR_VARIANT(128, 1, 2), PAIR_VARIANT(256, 2, 1), PAIR_VARIANT(256, 2, 2),
    // four
    QUAD_VARIANT(128, 1, 2), QUAD_VARIANT(256, 2, 2),
};
#undef TILE_VARIANT
#undef TILE8_VARIANT
#undef ONCE_VARIANT
#undef KG2_VARIANT
#undef KG2S_VARIANT
#undef WIDE_VARIANT
#undef WAVE_VARIANT
#undef PAIR_VARIANT
#undef QUAD_VARIANT
constexpr int N_VARIANTS = sizeof(VARIANTS) / sizeof(VARIANTS[0]);

// the variant a plan asks for, or nullptr
const Variant *find_variant(const dream_attn_desc *d, const Plan &p)
{
    const int family = !p.wave_mode ? FAMILY_TILE : p.slots == 1 ? FAMILY_WAVE : p.slots == 2 ? FAMILY_PAIR : FAMILY_QUAD;
    const int p1 = p.wave_mode ? p.wave_nw : p.qg, p2 = p.wave_mode ? p.wave_ds : p.kt, p3 = p.wave_mode ? p.wave_qt : p.pfd;
    const int p4 = p.wave_mode ? 0 : p.nw, p5 = p.wave_mode ? 1 : p.mw, p6 = p.wave_mode ? 0 : p.once, p7 = p.wave_mode ? 1 : p.kg;
    for (int i = 0; i < N_VARIANTS; i++) {
        const Variant &v = VARIANTS[i];
        if (v.family == family && v.d == d->head_dim && v.p1 == p1 && v.p2 == p2 && v.p3 == p3 && v.p4 == p4 && v.p5 == p5 && v.p6 == p6 && v.p7 == p7)
            return &v;
    }
    return nullptr;
}

void variant_name(const Variant &v, char *buf, size_t n)
{
    if (v.family == FAMILY_PAIR || v.family == FAMILY_QUAD)
        snprintf(buf, n, "attn_%s_kernel<%d,%d,%d>", v.family == FAMILY_PAIR ? "pair" : "quad", v.d, v.p2, v.p3);
    else if (v.family == FAMILY_WAVE)
        snprintf(buf, n, "attn_wave_kernel<%d,%d,%d,%d>", v.d, v.p1, v.p2, v.p3);
    else if (v.p7 != 1)
        snprintf(buf, n, "attn_bf16_kernel<%d,%d,%d,%d,%d,%d,%d,%d>", v.d, v.p1, v.p2, v.p3, v.p4, v.p5, v.p6, v.p7);
    else if (v.p6 && v.p4 == 4)
        snprintf(buf, n, "attn_bf16_kernel<%d,%d,%d,%d,%d,%d,%d>", v.d, v.p1, v.p2, v.p3, v.p4, v.p5, v.p6);
    else if (v.p5 != 1)
        snprintf(buf, n, "attn_bf16_kernel<%d,%d,%d,%d,%d,%d>", v.d, v.p1, v.p2, v.p3, v.p4, v.p5);
    else if (v.p4 != 4)
        snprintf(buf, n, "attn_bf16_kernel<%d,%d,%d,%d,%d>", v.d, v.p1, v.p2, v.p3, v.p4);
    else
        snprintf(buf, n, "attn_bf16_kernel<%d,%d,%d,%d>", v.d, v.p1, v.p2, v.p3);
}

// Bytes of keys and values from which on a call finds them in HBM and not in the 256 MB memory-side cache.  Verification reads every layer's caches once a round: from
// 8 MB a layer on the 24 to 48 layers of a model displace each other.  A draft's one cache is read again at the next level, and is still there while it fits beside
// the level's projection weights.
bool caches_near(const dream_attn_desc *d, int64_t max_kv_len, bool drafting)
{
    return (int64_t)d->batch * d->n_kv_heads * max_kv_len * d->head_dim * 4 < (int64_t)(drafting ? 152 : 8) << 20;
}

// AttnArgs::turn.  The orders in which most of a CU's keys have come to L2 before it asks for them pay while what the heads of an XCD have in flight stays there.
//
// RowsGeom::SWAPPED: always in a verification.  In a draft, whose caches come from the memory-side cache, only while the heads of an XCD fit its 4 MB L2 or nearly: 3 sequences of 32 heads,
// 10 rows, 1657 keys, 5.1 MB an XCD, us with the order / without: 10.1 / 9.5, 2233 keys 12.1 / 11.1; 4 sequences of 1145 keys, 4.7 MB, 7.4 / 7.7; a whole level of one sequence 9.4 / 9.6.
// RowsGeom::TURNED: with three workgroups to a KV head or more, up to 6 MB an XCD, and not in a draft (one sequence of 16 heads of 256, 1640 keys, 4 % more with it; 32 of 128 1 to 3 %).
// Verifications over 402 shapes (1 to 12 sequences, 17 to 60 rows, 250 to 2300 keys), us in lock step / with the order: head_dim 128, one sequence of 32 heads, 60 rows, 1340 keys 12.3 / 11.4, 1860 keys 15.9 / 14.8;
// 32 on 8 heads, 1 sequence of 60 rows, 2360 keys 17.3 / 15.2, 3 of 17 rows, 1297 keys 12.0 / 11.0; head_dim 256, 16 on 8 heads, 1 sequence of 60 rows, 1340 keys 16.8 / 15.5, 2 sequences 18.1 / 16.9, 4 of 33 rows, 5.4 MB,
// 20.5 / 20.2; head_dim 64, 2 sequences of 32 heads, 60 rows, 1860 keys 12.0 / 11.5.  On the other side: two workgroups to a head, 2 sequences of 32 heads of 128, 60 rows, 1340 keys, and the hint gone, 5 %
// slower; 6 of 16 on 8 heads of 256, 17 rows, 7 MB 6 %, 10 MB 16 %.  Two and three query tiles of head_dim 128, pairs and four slots, whose MFMAs take as long as the pull: 1 to 10 % slower, so they have no such order.
uint32_t order_of_tiles(const dream_attn_desc *d, const Plan &p, int n_q, int64_t max_kv_len, int verification)
{
    if (!p.wave_mode || p.slots != 1)
        return 0;
    const int64_t per_xcd = (int64_t)ceil_div((int64_t)d->batch * d->n_kv_heads, 8) * max_kv_len * d->head_dim * 4;
    const int workgroups = ceil_div(ceil_div((int64_t)(d->n_q_heads / d->n_kv_heads) * n_q, 16), p.wave_qt) * p.wave_ds;
    const bool swapped = d->head_dim == 64 && p.wave_ds == 2, turned = !swapped && (p.wave_qt == 1 || d->head_dim == 256);
    if ((swapped && (verification || per_xcd < 5000000)) || (turned && verification && workgroups >= 3 && per_xcd < 6000000))
        return (uint32_t)(TURN << 16) / workgroups;
    return 0;
}

int run_attention(const char *who, const dream_attn_desc *d, const void *q, const void *k, const void *v,
                  const int32_t *prefix_len, int n_tree, const int32_t *parent, const uint64_t *tree_mask,
                  int n_q, const int32_t *q_node, int include_self, int64_t max_kv_len, void *out, float *lse,
                  void *ws, size_t ws_bytes, void *stream)
{
    int rc = validate_desc(d, who);
    if (rc)
        return rc;
    if (!q || !k || !v || !prefix_len || !out)
        return fail(DREAM_ERR_INVALID_ARG, "%s: q, k, v, prefix_len and out must not be NULL", who);
    if (!parent && !tree_mask)
        return fail(DREAM_ERR_INVALID_ARG, "%s: parent is NULL and no tree_mask is given", who);
    if (n_tree < 1 || n_tree > DREAM_MAX_TREE)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: n_tree %d outside [1, %d]", who, n_tree, DREAM_MAX_TREE);
    if (n_q < 1 || n_q > DREAM_MAX_TREE)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: %d query rows outside [1, %d]", who, n_q, DREAM_MAX_TREE);
    if (!q_node && n_q > n_tree)
        return fail(DREAM_ERR_INVALID_ARG, "%s: %d query rows but only %d tree nodes and no q_node", who, n_q, n_tree);
    if (max_kv_len < n_tree || max_kv_len > d->s_max)
        return fail(DREAM_ERR_INVALID_ARG, "%s: max_kv_len %lld outside [n_tree, s_max]", who, (long long)max_kv_len);
    const bool direct = !((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k) | reinterpret_cast<uintptr_t>(v)) & 15);
    Plan p = {};
    // (unaligned tensors get what the workspace was asked for, never more splits than that)
    make_plan(d, n_q, max_kv_len, direct, caches_near(d, max_kv_len, !include_self && direct), &p);
    if (n_tree > 64 && d->dtype == DREAM_BF16)
        make_wide_plan(d, n_q, &p);
    if (!ws || ws_bytes < p.total)
        return fail(DREAM_ERR_WORKSPACE, "%s: workspace of %zu bytes, %zu needed", who, ws_bytes, p.total);

    AttnArgs a;
    a.q = q; a.k = k; a.v = v;
    a.prefix_len = prefix_len; a.parent = parent; a.q_node = q_node; a.tree_mask = tree_mask;
    a.out = out; a.lse = lse;
    a.part = reinterpret_cast<float *>(static_cast<char *>(ws) + p.off_part);
    a.n_q_heads = d->n_q_heads; a.n_kv_heads = d->n_kv_heads; a.group = d->n_q_heads / d->n_kv_heads;
    a.n_q = n_q; a.n_tree = n_tree; a.include_self = include_self;
    a.mask_words = ceil_div(n_tree, 64);
    a.n_qg = p.n_qg; a.n_splits = p.n_splits; a.n_streams = p.n_streams;
    auto magic = [](int x) { return x == 1 ? 0u : (uint32_t)(((1ull << 32) + x - 1) / x); };
    a.nq_magic = magic(n_q);
    a.spread = d->n_kv_heads % 8 ? (65536 + d->n_kv_heads - 1) / d->n_kv_heads : 0;
    // The nontemporal hint where the caches come from HBM: it keeps them from displacing the rows other workgroups still read (us with
    // plain loads / with the hint: 32 heads of head_dim 128 and 764 keys 8.97 / 8.73, 4 sequences of them 15.2 / 13.2; 8 sequences of 10 rows, head_dim 64, 20.1 / 17.8;
    // but 5.5 MB a layer 9.4 / 11.0; in 4 column slices, whose workgroups read a quarter of a V row each, head_dim 256, 4 sequences of 33 rows, 20.6 / 21.2: never).
    // (A whole LLaVA draft: 4 sequences, 110 MB 324 / 332, 147 MB 364 / 371; 8 sequences, 156 MB 441 / 424, 192 MB 482 / 422, 294 MB 633 / 544).
    a.once = !caches_near(d, max_kv_len, !include_self);
    if (p.wave_mode) {
        a.turn = order_of_tiles(d, p, n_q, max_kv_len, include_self);
        if (a.turn)
            a.once = 0;      // (a row that goes back into L2 as the first to leave is not found there)
    } else {
        a.tiles_per_head = p.tiles_per_head;
    }
    a.s_max = d->s_max;
    a.scale = d->scale != 0.0f ? d->scale : 1.0f / sqrtf((float)d->head_dim);
    a.scale_log2 = a.scale * 1.4426950408889634f;
    hipStream_t st = as_stream(stream);

    if (d->dtype == DREAM_F32) {
        dim3 grid(n_q, d->n_q_heads, d->batch);
        hipLaunchKernelGGL(d->head_dim == 64 ? attn_f32_kernel<64> : d->head_dim == 128 ? attn_f32_kernel<128> : attn_f32_kernel<256>, grid, dim3(256),
                           0, st, a);
        return check_launch("attn_f32_kernel");
    }

    const Variant *variant = find_variant(d, p);
    if (!variant)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: no kernel variant for head_dim %d with launch parameters (%d, %d, %d)", who, d->head_dim,
                    p.wave_mode ? p.wave_nw : p.qg, p.wave_mode ? p.wave_ds : p.kt, p.wave_mode ? p.wave_qt : p.pfd);
    if (p.wave_mode && (n_tree > 64 || a.group > 4 || a.group * n_q > 16 * 16 || p.n_streams > 256))
        return fail(DREAM_ERR_UNSUPPORTED, "%s: the plan names a kernel that cannot serve %d streams of %d rows", who, p.n_streams, a.group * n_q);
    return variant->launch(a, p, st);
}

size_t workspace_for(const dream_attn_desc *d, int n_q, int64_t max_kv_len)
{
    if (!d || d->n_kv_heads < 1 || d->n_q_heads < 1 || d->n_q_heads % d->n_kv_heads || n_q < 1 || max_kv_len < 1 ||
        d->batch < 1)
        return DREAM_WORKSPACE_MIN_BYTES;
    Plan p = {};
    make_plan(d, n_q, max_kv_len, true, caches_near(d, max_kv_len, false), &p);
    return p.total;
}

}  // namespace

namespace dream {
// every attention kernel variant the launch plan can choose (part of dream_init)
int attn_init()
{
    for (int i = 0; i < N_VARIANTS; i++)
        if (int rc = VARIANTS[i].ensure())
            return rc;
    return DREAM_OK;
}
}  // namespace dream

extern "C" {

int dream_attn_plan_describe(const dream_attn_desc *desc, int32_t n_q, int64_t max_kv_len, char *buf, size_t buf_bytes)
{
    const char *who = "dream_attn_plan_describe";
    if (!buf || buf_bytes == 0)
        return fail(DREAM_ERR_INVALID_ARG, "%s: no buffer", who);
    int rc = validate_desc(desc, who);
    if (rc)
        return rc;
    if (n_q < 1 || max_kv_len < 1 || max_kv_len > desc->s_max)
        return fail(DREAM_ERR_INVALID_ARG, "%s: need n_q >= 1 and 1 <= max_kv_len <= s_max", who);
    Plan p = {};
    make_plan(desc, n_q, max_kv_len, true, caches_near(desc, max_kv_len, false), &p);
    if (n_q > 64 && desc->dtype == DREAM_BF16)   // more than 64 query rows: taken as a verification call over a tree of n_q nodes
        make_wide_plan(desc, n_q, &p);
    if (desc->dtype == DREAM_F32) {
        snprintf(buf, buf_bytes, "attn_f32_kernel workgroups=%lld", (long long)desc->batch * desc->n_q_heads * n_q);
        return DREAM_OK;
    }
    const Variant *v = find_variant(desc, p);
    if (!v)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: the plan names a kernel variant that is not built", who);
    char name[64];
    variant_name(*v, name, sizeof name);
    if (p.wave_mode)
        snprintf(buf, buf_bytes, "%s workgroups=%d splits=1 merge_launch=0", name,
                 ceil_div(p.n_qg, p.slots * p.wave_qt) * p.wave_ds * desc->n_kv_heads * desc->batch);
    else
        snprintf(buf, buf_bytes, "%s workgroups=%d splits=%d merge_launch=%d", name, p.n_groups * p.n_splits, p.n_splits,
                 p.n_splits > 1 ? 1 : 0);
    return DREAM_OK;
}

int dream_attn_variants(char *buf, size_t buf_bytes)
{
    if (!buf || buf_bytes == 0)
        return fail(DREAM_ERR_INVALID_ARG, "dream_attn_variants: no buffer");
    size_t used = 0;
    buf[0] = 0;
    for (int i = 0; i < N_VARIANTS; i++) {
        char name[64];
        variant_name(VARIANTS[i], name, sizeof name);
        const int n = snprintf(buf + used, buf_bytes - used, "%s%s", i ? ";" : "", name);
        if (n < 0 || (size_t)n >= buf_bytes - used)
            return fail(DREAM_ERR_INVALID_ARG, "dream_attn_variants: buffer of %zu bytes is too small", buf_bytes);
        used += (size_t)n;
    }
    return DREAM_OK;
}

size_t dream_tree_verify_attn_workspace(const dream_attn_desc *desc, int32_t n_tree, int64_t max_kv_len)
{
    return workspace_for(desc, n_tree, max_kv_len);
}

int dream_tree_verify_attn(const dream_attn_desc *desc, const void *q, const void *k_cache, const void *v_cache,
                           const int32_t *prefix_len, int32_t n_tree, const int32_t *parent,
                           const uint64_t *tree_mask, int64_t max_kv_len, void *out, float *lse,
                           void *workspace, size_t workspace_bytes, void *stream)
{
    return run_attention("dream_tree_verify_attn", desc, q, k_cache, v_cache, prefix_len, n_tree, parent, tree_mask,
                         n_tree, nullptr, 1, max_kv_len, out, lse, workspace, workspace_bytes, stream);
}

size_t dream_draft_xattn_workspace(const dream_attn_desc *desc, int32_t n_q, int64_t max_kv_len)
{
    return workspace_for(desc, n_q, max_kv_len);
}

int dream_draft_xattn(const dream_attn_desc *desc, const void *q, const void *kx_cache, const void *vx_cache,
                      const int32_t *prefix_len, int32_t n_tree, const int32_t *parent, int32_t n_q,
                      const int32_t *q_node, int64_t max_kv_len, void *out, void *workspace,
                      size_t workspace_bytes, void *stream)
{
    if (!parent)
        return fail(DREAM_ERR_INVALID_ARG, "dream_draft_xattn: parent must not be NULL");
    return run_attention("dream_draft_xattn", desc, q, kx_cache, vx_cache, prefix_len, n_tree, parent, nullptr,
                         n_q, q_node, 0, max_kv_len, out, nullptr, workspace, workspace_bytes, stream);
}

}  // extern "C"
