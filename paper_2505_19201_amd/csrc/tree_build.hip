// Draft-tree construction (Section 3.1, last paragraph: width-k tree expansion with the top-k reordering of
// EAGLE-2; Section 4: k children per node, a depth, a maximum number of drafted tokens).
//
// dream_tree_expand_level  one level of the expansion: for every frontier node the log-softmax of its draft
//   logits, its k most probable tokens as candidate children with score = score(node) + log p(token | node),
//   and the k best candidates of the level as the next frontier.
//     expand_partial_kernel  one workgroup per 8192-logit chunk of a row: the chunk is read once (16-byte
//       loads) into registers; it leaves the chunk's maximum and sum of exponentials and its k largest logits: the
//       elements at or above a lower bound of the k-th are collected in LDS and ranked by counting (k rounds of a
//       block-wide arg-max where ties make them too many).  The order is (logit descending, token
//       ascending) and compares the logits themselves, so the chosen tokens are exact whatever the chunking.
//     expand_merge_kernel    one workgroup per sequence, one wave per frontier row: merges the chunk partials
//       (log-sum-exp; the chunk candidates above a lower bound of the k-th ranked by counting), writes tokens and scores, then
//       ranks the F*k candidates by counting (score descending, index ascending) for the next frontier.
// dream_tree_finalize  the root and the `budget` best candidates of all levels, in creation order, parents
//   re-indexed: one wave finds the last kept score bit by bit and numbers the kept entries with ballots.
// Roofline: the expansion is an HBM scan of B*F*V logits (launch-latency bound at one sequence); the rest is
// latency bound by construction (a few hundred candidates).
#include "common.h"

using namespace dream;

namespace {

constexpr int CHUNK = 8192;          // logits per workgroup of the partial kernel
constexpr int PER_THREAD = CHUNK / 256;
constexpr int PAD = 8;               // keys counted at a time
constexpr int MAX_K = 16;            // DREAM_MAX_TREE_WIDTH
constexpr int MAX_F = 16;            // frontier rows per sequence (one wave each in the merge kernel)

// (value, index) pairs are ranked as one 64-bit key: the float mapped to an unsigned integer with the same
// order in the high word, the complemented index in the low word, so a larger key is a larger value or, among
// equal values, a lower index.  One integer compare per candidate instead of a float/integer cascade.
__device__ __forceinline__ uint32_t order_bits(float x)
{
    x += 0.0f;   // -0 and +0 are equal values: give them one key
    const uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float value_of(uint32_t k) { return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k); }
__device__ __forceinline__ uint64_t make_key(float v, int i) { return ((uint64_t)order_bits(v) << 32) | (uint32_t)(0xffffffffu - (uint32_t)i); }
__device__ __forceinline__ int index_of(uint64_t k) { return (int)(0xffffffffu - (uint32_t)k); }

// Maximum of a 64-bit key over the wave, returned in every lane.  Inside each row of 16 lanes the key is
// combined with its rotations by 8, 4, 2 and 1 lanes (DPP row_ror: a VALU move, no LDS round trip), which
// leaves the row maximum in all 16 lanes; the four row maxima are then read as scalars.
template <int ROT>
__device__ __forceinline__ uint64_t row_rotate_u64(uint64_t k)
{
    constexpr int ctrl = 0x120 + ROT;   // DPP row_ror:ROT
    const uint32_t lo = __builtin_amdgcn_update_dpp(0u, (uint32_t)k, ctrl, 0xf, 0xf, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0u, (uint32_t)(k >> 32), ctrl, 0xf, 0xf, false);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t lane_value(uint64_t k, int lane)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(k >> 32), lane) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)k, lane);
}
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t k)
{
    uint64_t o = row_rotate_u64<8>(k);
    k = o > k ? o : k;
    o = row_rotate_u64<4>(k);
    k = o > k ? o : k;
    o = row_rotate_u64<2>(k);
    k = o > k ? o : k;
    o = row_rotate_u64<1>(k);
    k = o > k ? o : k;
    const uint64_t a = lane_value(k, 0), b = lane_value(k, 16), c = lane_value(k, 32), d = lane_value(k, 48);
    const uint64_t ab = a > b ? a : b, cd = c > d ? c : d;
    return ab > cd ? ab : cd;
}

// What bounds it is latency, not bytes (one LLaVA level is 0.6 MB): the chunk is read once, and between the loads and the
// stores there are two barriers and no cross-lane exchange through LDS.  10 rows of 32000 bf16 logits: 7.0 -> 6.7 us, 80 rows of 49152 7.7 -> 7.1,
// since a wave places its candidates by ballot (each one's LDS atomic before was waited for).
// A call of both kernels, loads under conditions for the end of a row, each waited for before the next / all loads at once: 10 rows of 32000 bf16 10.8 / 9.8 us, 80 of 49152
// 12.7 / 11.7, 10 of 262144 13.2 / 12.2, 10 of 32000 float32 10.9 / 10.0; rows of odd lengths one logit at a time / in pieces off their boundaries: 10 of 32003 bf16 12.6 / 11.2,
// 80 of 50257 float32 24.0 / 22.8.
template <bool BF16>
__global__ __launch_bounds__(256) void expand_partial_kernel(const void *logits, int vocab, int n_chunks, int k, float *part_m,
                                                             float *part_s, uint64_t *part_key)
{
    __shared__ float s_f[4];
    __shared__ uint64_t s_k[4];
    const int chunk = blockIdx.x;
    const int64_t row = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint64_t below = (1ull << lane) - 1ull;
    const int begin = chunk * CHUNK;
    // element e of this thread is token begin + (e / 8) * 2048 + tid * 8 + e % 8.  Whole groups of 8 come in 16-byte loads, which global memory serves from any address of a logit (rows
    // of an odd vocabulary start anywhere), the rest one by one.  All are asked for before the first is waited for, so there is no load under a condition: what lies past
    // the end is another's and turned into -inf.
    float x[PER_THREAD];
    constexpr int ESZ = BF16 ? 2 : 4, W = BF16 ? 1 : 2;   // bytes of a logit, 16-byte pieces of a group
    const char *p = reinterpret_cast<const char *>(logits) + (row * vocab + begin) * ESZ;
    const int n_here = min(CHUNK, vocab - begin), n_groups = n_here / 8;
    auto one = [&](int t) { return BF16 ? bf16_bits_to_float(reinterpret_cast<const uint16_t *>(p)[t]) : reinterpret_cast<const float *>(p)[t]; };
    if (n_groups > 0) {
        u32x4 w[PER_THREAD / 8][W];
#pragma unroll
        for (int j = 0; j < PER_THREAD / 8; j++)
#pragma unroll
            for (int i = 0; i < W; i++) {
                const u32x4_any *from = reinterpret_cast<const u32x4_any *>(p) + min(j * 256 + tid, n_groups - 1) * W + i;
                w[j][i] = BF16 ? __builtin_nontemporal_load(from) : *from;     // bf16 logits: read once
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < PER_THREAD; e++) {
            const int j = e / 8, q = e % 8;
            x[e] = __uint_as_float(!BF16 ? w[j][q / 4 % W][q % 4] : q & 1 ? w[j][0][q / 2] & 0xffff0000u : w[j][0][q / 2] << 16);
        }
    }
    if (n_groups < CHUNK / 8) {
#pragma unroll
        for (int e = 0; e < PER_THREAD; e++)
            x[e] = e / 8 * 256 + tid < n_groups ? x[e] : -INFINITY;
        if (n_here % 8) {                                                      // the last group is no whole one
#pragma unroll
            for (int j = 0; j < PER_THREAD / 8; j++)
                if (j * 256 + tid == n_groups)
#pragma unroll
                    for (int q = 0; q < 8; q++)
                        x[j * 8 + q] = q < n_here % 8 ? one(min(n_groups * 8 + q, n_here - 1)) : -INFINITY;
        }
    }

    // ---- the 256 thread maxima fall into 16 rows of 16 lanes.  Their maximum is the chunk's, and the k-th largest of the 16 row
    // maxima is a lower bound of the chunk's k-th largest logit (at least k elements are at or above it).  Every wave ranks
    // the 16 for itself.
    __shared__ __attribute__((aligned(16))) float s_row[16];
    __shared__ int s_count[4];
    __shared__ __attribute__((aligned(16))) uint64_t s_cand[4][256 + PAD];
    float m = -INFINITY;
#pragma unroll
    for (int e = 0; e < PER_THREAD; e++)
        m = fmaxf(m, x[e]);                              // (padding is -inf)
    m = row_max(m);
    if ((lane & 15) == 0)
        s_row[tid >> 4] = m;
    __syncthreads();
    float rows[16];
#pragma unroll
    for (int j = 0; j < 16; j++)
        rows[j] = s_row[j];
    const float mine = s_row[lane & 15];
    int row_rank = 0;
    m = rows[0];
#pragma unroll
    for (int j = 0; j < 16; j++) {
        row_rank += (rows[j] > mine || (rows[j] == mine && j < (lane & 15))) ? 1 : 0;
        m = fmaxf(m, rows[j]);
    }
    const float tau = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), __builtin_ctzll(__ballot(row_rank == min(k, 16) - 1))));
    // sum of exponentials relative to the maximum
    const float base = m == -INFINITY ? 0.0f : m;        // (a chunk of -inf only sums to 0)
    float s = 0.0f;
#pragma unroll
    for (int e = 0; e < PER_THREAD; e++)
        s += __expf(x[e] - base);
    s = wave_sum(s);
    // ---- the chunk's k largest: the elements at or above the bound (a few dozen for ordinary logits) are collected in LDS, each
    // wave's by itself, and ranked by counting; more than 256 of them (heavy ties) fall back to k rounds of a block-wide arg-max.
    int n_mine = 0;                                      // of this wave
#pragma unroll
    for (int e = 0; e < PER_THREAD; e++) {
        const uint64_t hits = __ballot(x[e] >= tau);
        if (hits != 0) {
            const int t = begin + (e >> 3) * 2048 + tid * 8 + (e & 7);
            const bool hit = x[e] >= tau && t < vocab;   // (a bound of -inf also takes the padding)
            const uint64_t take = __ballot(hit);
            const int slot = n_mine + __popcll(take & below);
            if (hit && slot < 256)
                s_cand[wave][slot] = make_key(x[e], t);
            n_mine += __popcll(take);
        }
    }
    if (lane < PAD && n_mine <= 256)                     // zeros rank below every key: the counting takes PAD keys at a time
        s_cand[wave][n_mine + lane] = 0ull;
    if (lane == 0) {
        s_f[wave] = s;
        s_count[wave] = n_mine;
    }
    __syncthreads();
    if (tid == 0) {
        part_m[row * n_chunks + chunk] = m;
        part_s[row * n_chunks + chunk] = (s_f[0] + s_f[1]) + (s_f[2] + s_f[3]);
    }
    const int n0 = s_count[0], n1 = n0 + s_count[1], n2 = n1 + s_count[2], n_cand = n2 + s_count[3];
    uint64_t *out_key = part_key + (row * n_chunks + chunk) * k;
    if (n_cand <= 256) {
        if (tid < n_cand) {
            const int from = (tid >= n0) + (tid >= n1) + (tid >= n2);
            const uint64_t mine = s_cand[from][tid - (from == 0 ? 0 : from == 1 ? n0 : from == 2 ? n1 : n2)];
            int rank = 0;
#pragma unroll
            for (int w = 0; w < 4; w++) {
                const int n = s_count[w];
                for (int j = 0; j < n; j += PAD)
#pragma unroll
                    for (int i = 0; i < PAD; i++)
                        rank += s_cand[w][j + i] > mine ? 1 : 0;
            }
            if (rank < k)
                out_key[rank] = mine;
        }
        if (tid >= n_cand && tid < k)
            out_key[tid] = 0ull;   // fewer than k tokens in the chunk
        return;
    }
    // keys of this thread's elements (0 for tokens past the vocabulary: below every real key)
    uint64_t key[PER_THREAD];
#pragma unroll
    for (int e = 0; e < PER_THREAD; e++) {
        const int t = begin + (e >> 3) * 2048 + tid * 8 + (e & 7);
        key[e] = t < vocab ? make_key(x[e], t) : 0ull;
    }
    // k rounds: the largest key below the previous pick
    uint64_t prev = ~0ull;
    for (int r = 0; r < k; r++) {
        uint64_t best = 0ull;
#pragma unroll
        for (int e = 0; e < PER_THREAD; e++) {
            const uint64_t c = key[e] < prev ? key[e] : 0ull;
            best = c > best ? c : best;
        }
        best = wave_max_u64(best);
        if (lane == 0)
            s_k[wave] = best;
        __syncthreads();
        best = s_k[0];
#pragma unroll
        for (int w = 1; w < 4; w++)
            best = s_k[w] > best ? s_k[w] : best;
        __syncthreads();
        if (tid == 0)
            out_key[r] = best;   // 0 once the chunk is exhausted
        prev = best;
    }
}

// One workgroup per sequence; wave f merges the chunk partials of frontier row f.  PART: chunk candidates a lane
// holds (1, 2, 4 or 8).  Latency bound: every load of a row is issued before the first result is needed, and four waves share a
// SIMD, so instructions count: k rounds of a wave arg-max over all candidates, one lane writing, took 6.1 us at 10 rows and k = 10, ranking the
// few above a bound of the k-th 4.5 (one row 4.2 -> 3.5; drafting 6 levels: LLaVA 233 -> 223 us, 8 SmolVLM sequences 273 -> 263).
// bound: ceil(k / chunks) and, from bit 8 on, ceil(k / that), which were divisions ahead of the loads; with up to 64 chunks one load of their sums a lane instead of eight conditions: drafts 202.5 -> 200.5
// and 231.9 -> 229.6 us.
template <int PART>
__global__ __launch_bounds__(64 * MAX_F) void expand_merge_kernel(const float *part_m, const float *part_s, const uint64_t *part_key,
                                                                  int n_frontier, int n_chunks, int k, int bound, const float *cum_in,
                                                                  int32_t *cand_token, float *cand_score, int32_t *next_frontier)
{
    __shared__ uint64_t s_key[MAX_F * MAX_K];   // (score, flat index) keys of the level's candidates
    __shared__ __attribute__((aligned(16))) uint64_t s_left[MAX_F][64 + PAD];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const uint64_t below = (1ull << lane) - 1ull;
    const int f = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_cand = n_frontier * k;
    if (f < n_frontier) {
        const int64_t row = (int64_t)b * n_frontier + f;
        const int n_part = n_chunks * k;
        uint64_t pk[PART];
#pragma unroll
        for (int j = 0; j < PART; j++)
            pk[j] = lane + j * 64 < n_part ? part_key[row * n_part + lane + j * 64] : 0ull;
        const int depth = bound & 0xff, q = bound >> 8;       // ceil(k / chunks), ceil(k / depth)
        // A few rounds cost less than the bound, whose chunks are counted one by one.  us, a level of 1 row / 10 rows, rounds and bound: 262144 tokens, k = 1 6.9 and 8.6 / 8.7 and
        // 10.8, k = 4 8.1 and 8.9 / 9.6 and 10.1; 131072 tokens, 10 rows, k = 1 7.7 and 8.7, k = 3 9.0 and 9.3, k = 4 9.3 and 9.3; 32000 tokens, 10 rows, k = 2 8.4 and 8.6, k = 3 9.0 and 8.7.
        const bool bounded = n_chunks <= 64 && k > 2 + n_chunks / 16;
        const uint64_t deep = bounded && lane < n_chunks ? part_key[row * n_part + lane * k + depth - 1] : 0ull;
        // log-sum-exp of the row from the chunk partials (8 per lane: with k = 1 there may be 512 chunks)
        float M = -INFINITY, cm[8], cs[8];
        const float cum = cum_in[row];
        const bool many = n_chunks > 64;
        cm[0] = lane < n_chunks ? part_m[row * n_chunks + lane] : -INFINITY;
        cs[0] = lane < n_chunks ? part_s[row * n_chunks + lane] : 0.0f;
#pragma unroll
        for (int j = 1; j < 8; j++) {
            cm[j] = -INFINITY;
            cs[j] = 0.0f;
        }
        if (many) {
#pragma unroll
            for (int j = 1; j < 8; j++) {
                const int ch = min(lane + j * 64, n_chunks - 1);
                cm[j] = part_m[row * n_chunks + ch];
                cs[j] = part_s[row * n_chunks + ch];
            }
#pragma unroll
            for (int j = 1; j < 8; j++)
                cm[j] = lane + j * 64 < n_chunks ? cm[j] : -INFINITY;
        }
#pragma unroll
        for (int j = 0; j < 8; j++)
            M = fmaxf(M, cm[j]);
        M = wave_max(M);
        float S = cm[0] == -INFINITY ? 0.0f : cs[0] * __expf(cm[0] - M);
        if (many)
#pragma unroll
            for (int j = 1; j < 8; j++)
                S += cm[j] == -INFINITY ? 0.0f : cs[j] * __expf(cm[j] - M);
        S = wave_sum(S);
        const float lse = M + __logf(S);
        auto emit = [&](int r, uint64_t best) {
            const float sc = cum + (value_of((uint32_t)(best >> 32)) - lse);
            cand_token[row * k + r] = index_of(best);
            cand_score[row * k + r] = sc;
            s_key[f * k + r] = make_key(sc, f * k + r);
        };
        // A lower bound of the k-th key: with q = ceil(k / depth) chunks whose depth-th key is at or above it there are k keys
        // at or above it.  Lane c holds the depth-th of chunk c; the q-th of those is found by counting.
        int n_left = 65;
        if (bounded) {
            int above = 0;
            for (int c = 0; c < n_chunks; c++)
                above += lane_value(deep, c) > deep ? 1 : 0;
            const uint64_t at = __ballot(lane < n_chunks && above == q - 1);
            uint64_t tau = at ? lane_value(deep, __builtin_ctzll(at)) : 0ull;
            tau = tau ? tau : 1ull;                       // (0 is no token)
            n_left = 0;
#pragma unroll
            for (int j = 0; j < PART; j++) {
                const bool keep = pk[j] >= tau;
                const uint64_t take = __ballot(keep);
                const int slot = n_left + __popcll(take & below);
                if (keep && slot < 64)
                    s_left[f][slot] = pk[j];
                n_left += __popcll(take);
            }
        }
        if (n_left <= 64) {                               // the rule: 10 to 30 keys, one per lane, ranked by counting
            if (lane < PAD)
                s_left[f][n_left + lane] = 0ull;
            wave_lds_fence();
            const uint64_t mine = lane < n_left ? s_left[f][lane] : 0ull;
            int rank = lane < n_left ? 0 : lane;
            for (int j = 0; j < n_left; j += PAD)
#pragma unroll
                for (int i = 0; i < PAD; i++)
                    rank += lane < n_left && s_left[f][j + i] > mine ? 1 : 0;
            if (rank < k)
                emit(rank, mine);
        } else {                                          // k rounds: the largest key below the previous pick
            uint64_t prev = ~0ull;
            for (int r = 0; r < k; r++) {
                uint64_t best = 0ull;
#pragma unroll
                for (int j = 0; j < PART; j++) {
                    const uint64_t c = pk[j] < prev ? pk[j] : 0ull;
                    best = c > best ? c : best;
                }
                best = wave_max_u64(best);
                if (lane == 0)
                    emit(r, best);
                prev = best;
            }
        }
    }
    __syncthreads();
    // next frontier: rank of every candidate = number of larger keys; 4 threads share a candidate
    const int kf = min(k, n_cand);
    const int cand = tid >> 2, part = tid & 3;
    int rank = 0;
    if (cand < n_cand) {
        const uint64_t mine = s_key[cand];
#pragma unroll 8
        for (int j = part; j < n_cand; j += 4)
            rank += s_key[j] > mine ? 1 : 0;
    }
    rank += __shfl_xor(rank, 1);
    rank += __shfl_xor(rank, 2);
    if (cand < n_cand && part == 0 && rank < kf)
        next_frontier[(int64_t)b * kf + rank] = cand;
}

// One wave per sequence, the whole pool in its registers (entry r * 64 + lane in register r), so nothing has to be
// synchronised: the score of the last kept entry is found bit by bit, counting entries at or above a trial value with a compare
// and a population count per register, and stops as soon as a trial value keeps exactly the asked number.  (Ranking
// every entry by counting larger ones took 10.7 us for a pool of 511: a quarter of a million compares fed from LDS.)
template <int NR>
__global__ __launch_bounds__(64) void tree_finalize_kernel(const float *pool_score, const int32_t *pool_parent, const int32_t *pool_token,
                                                           int n_pool, int keep_n, int32_t *tree_parent, int32_t *tree_token,
                                                           int32_t *tree_pool_index)
{
    __shared__ int32_t s_new[NR * 64];          // new index of a kept entry, -2 for a dropped one
    const int b = blockIdx.x, lane = threadIdx.x;
    const int64_t at = (int64_t)b * n_pool;
    float sc[NR];
    uint32_t key[NR];
    int32_t par[NR], tok[NR];
#pragma unroll
    for (int r = 0; r < NR; r++) {
        const int64_t i = at + min(r * 64 + lane, n_pool - 1);   // (unconditional loads: all in flight together)
        sc[r] = pool_score[i];
        par[r] = pool_parent[i];
        tok[r] = pool_token[i];
    }
#pragma unroll
    for (int r = 0; r < NR; r++) {
        const int i = r * 64 + lane;
        key[r] = i > 0 && i < n_pool ? max(order_bits(sc[r]), 1u) : 0u;    // (0 is no entry: the NaN of all ones would have it too)
    }
    // the largest value with at least keep_n entries at or above it
    uint32_t cut = 0u;
    int at_cut = -1;                              // entries at or above `cut`
#pragma unroll 1
    for (int bit = 31; bit >= 0 && keep_n > 0; bit--) {
        const uint32_t trial = cut | (1u << bit);
        int n = 0;
#pragma unroll
        for (int r = 0; r < NR; r++)
            n += __popcll(__ballot(key[r] >= trial));
        if (n >= keep_n) {
            cut = trial;
            at_cut = n;
            if (n == keep_n)
                break;
        }
    }
    // with more entries than asked for, those at the cut itself are kept in index order
    int spare = 0x7fffffff;
    if (at_cut > keep_n) {
        int above = 0;
#pragma unroll
        for (int r = 0; r < NR; r++)
            above += __popcll(__ballot(key[r] > cut));
        spare = keep_n - above;
    }
    const uint64_t below = (1ull << lane) - 1ull;
    int base = 0;
    bool keep[NR];
#pragma unroll
    for (int r = 0; r < NR; r++) {
        const bool tie = keep_n > 0 && key[r] == cut && key[r] != 0u;
        const uint64_t ties = __ballot(tie);
        const bool take_tie = tie && (int)__popcll(ties & below) < spare;
        keep[r] = (r == 0 && lane == 0) || (keep_n > 0 && key[r] > cut) || take_tie;
        spare -= (int)__popcll(ties);
        const uint64_t kept = __ballot(keep[r]);
        s_new[r * 64 + lane] = keep[r] ? base + __popcll(kept & below) : -2;
        base += __popcll(kept);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; r++)
        if (keep[r]) {
            const int64_t o = (int64_t)b * (1 + keep_n) + s_new[r * 64 + lane];
            tree_parent[o] = r == 0 && lane == 0 ? -1 : ((par[r] >= 0 && par[r] < n_pool) ? s_new[par[r]] : -2);
            tree_token[o] = tok[r];
            tree_pool_index[o] = r * 64 + lane;
        }
}

struct ExpandPlan {
    int n_chunks;
    size_t off_m, off_s, off_key, total;
};

ExpandPlan expand_plan(int batch, int n_frontier, int vocab, int k)
{
    ExpandPlan p;
    p.n_chunks = ceil_div(vocab, CHUNK);
    const size_t rows = (size_t)batch * n_frontier;
    p.off_m = DREAM_WORKSPACE_MIN_BYTES;
    p.off_s = align_up(p.off_m + rows * p.n_chunks * sizeof(float), 256);
    p.off_key = align_up(p.off_s + rows * p.n_chunks * sizeof(float), 256);
    p.total = align_up(p.off_key + rows * p.n_chunks * k * sizeof(uint64_t), 256);
    return p;
}

}  // namespace

extern "C" {

size_t dream_tree_expand_workspace(int32_t batch, int32_t n_frontier, int32_t vocab, int32_t k)
{
    if (batch < 1 || n_frontier < 1 || vocab < 1 || k < 1)
        return DREAM_WORKSPACE_MIN_BYTES;
    return expand_plan(batch, n_frontier, vocab, k).total;
}

int dream_tree_expand_level(const void *logits, int32_t logits_dtype, int32_t batch, int32_t n_frontier, int32_t vocab,
                            const float *cum_in, int32_t k, int32_t *cand_token, float *cand_score, int32_t *next_frontier,
                            void *workspace, size_t workspace_bytes, void *stream)
{
    const char *who = "dream_tree_expand_level";
    if (!logits || !cum_in || !cand_token || !cand_score || !next_frontier)
        return fail(DREAM_ERR_INVALID_ARG, "%s: NULL argument", who);
    if (logits_dtype != DREAM_F32 && logits_dtype != DREAM_BF16)
        return fail(DREAM_ERR_INVALID_ARG, "%s: unknown dtype %d", who, logits_dtype);
    if (batch < 1 || batch > 65535)
        return fail(DREAM_ERR_INVALID_ARG, "%s: batch %d outside [1, 65535]", who, batch);
    if (n_frontier < 1 || n_frontier > MAX_F)
        return fail(DREAM_ERR_INVALID_ARG, "%s: n_frontier %d outside [1, %d]", who, n_frontier, MAX_F);
    if (k < 1 || k > DREAM_MAX_TREE_WIDTH || k > vocab)
        return fail(DREAM_ERR_INVALID_ARG, "%s: k %d outside [1, min(%d, vocab)]", who, k, DREAM_MAX_TREE_WIDTH);
    if (ceil_div(vocab, CHUNK) * k > 64 * 8)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: vocab %d with k %d exceeds the 512 chunk candidates a wave merges", who, vocab, k);
    if (vocab < 1 || (int64_t)batch * n_frontier > 65535)
        return fail(DREAM_ERR_INVALID_ARG, "%s: vocab must be positive and batch * n_frontier at most 65535", who);
    ExpandPlan p = expand_plan(batch, n_frontier, vocab, k);
    if (!workspace || workspace_bytes < p.total)
        return fail(DREAM_ERR_WORKSPACE, "%s: workspace of %zu bytes, %zu needed", who, workspace_bytes, p.total);
    char *ws = static_cast<char *>(workspace);
    float *pm = reinterpret_cast<float *>(ws + p.off_m), *ps = reinterpret_cast<float *>(ws + p.off_s);
    uint64_t *pkey = reinterpret_cast<uint64_t *>(ws + p.off_key);
    hipStream_t st = as_stream(stream);
    const dim3 grid(p.n_chunks, batch * n_frontier);
    if (logits_dtype == DREAM_BF16)
        hipLaunchKernelGGL(expand_partial_kernel<true>, grid, dim3(256), 0, st, logits, vocab, p.n_chunks, k, pm, ps, pkey);
    else
        hipLaunchKernelGGL(expand_partial_kernel<false>, grid, dim3(256), 0, st, logits, vocab, p.n_chunks, k, pm, ps, pkey);
    int rc = check_launch("expand_partial_kernel");
    if (rc)
        return rc;
    const int n_part = p.n_chunks * k;
    auto merge = n_part <= 64 ? expand_merge_kernel<1> : n_part <= 128 ? expand_merge_kernel<2> : n_part <= 256 ? expand_merge_kernel<4> : expand_merge_kernel<8>;
    const int depth = ceil_div(k, p.n_chunks), bound = depth | ceil_div(k, depth) << 8;
    hipLaunchKernelGGL(merge, dim3(batch), dim3(64 * n_frontier), 0, st, pm, ps, pkey, n_frontier, p.n_chunks, k, bound, cum_in, cand_token, cand_score, next_frontier);
    return check_launch("expand_merge_kernel");
}

int dream_tree_finalize(const float *pool_score, const int32_t *pool_parent, const int32_t *pool_token, int32_t batch, int32_t n_pool,
                        int32_t budget, int32_t *tree_parent, int32_t *tree_token, int32_t *tree_pool_index, int32_t *n_tree_host,
                        void *stream)
{
    const char *who = "dream_tree_finalize";
    if (!pool_score || !pool_parent || !pool_token || !tree_parent || !tree_token || !tree_pool_index)
        return fail(DREAM_ERR_INVALID_ARG, "%s: NULL argument", who);
    if (batch < 1 || batch > 65535)
        return fail(DREAM_ERR_INVALID_ARG, "%s: batch %d outside [1, 65535]", who, batch);
    if (n_pool < 1 || n_pool > DREAM_MAX_POOL)
        return fail(DREAM_ERR_INVALID_ARG, "%s: n_pool %d outside [1, %d]", who, n_pool, DREAM_MAX_POOL);
    if (budget < 0)
        return fail(DREAM_ERR_INVALID_ARG, "%s: negative budget", who);
    const int keep_n = budget < n_pool - 1 ? budget : n_pool - 1;
    if (n_tree_host)
        *n_tree_host = 1 + keep_n;
    auto kernel = n_pool <= 128 ? tree_finalize_kernel<2> : n_pool <= 256 ? tree_finalize_kernel<4> : n_pool <= 512 ? tree_finalize_kernel<8> : tree_finalize_kernel<16>;
    hipLaunchKernelGGL(kernel, dim3(batch), dim3(64), 0, as_stream(stream), pool_score, pool_parent, pool_token, n_pool, keep_n, tree_parent,
                       tree_token, tree_pool_index);
    return check_launch("tree_finalize_kernel");
}

}  // extern "C"
