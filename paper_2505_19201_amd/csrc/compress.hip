// dream_visual_compress: visual-token importance scores, top-k keep and row gather (Section 3.3).
//
// The importance of key token j is the attention weight it receives, summed over the rows and
// heads of the last-layer causal attention matrix.  The probabilities need each row's softmax
// normaliser first, so stage A runs two passes over q k^T on the matrix cores, no attention matrix is ever stored:
//   scores_lse_*     one workgroup per 64 or 128 query rows, K streamed through LDS, tiles of 32x32: log-sum-exp of every causal row;
//   scores_colsum_*  one workgroup per 64 or 128 visual keys, query rows streamed through LDS, tiles of 16x16: sum over rows of
//                    exp(score - lse), per head.
// Every (sequence, head, row split, key) partial sum has one fixed order of additions, and the selection kernel adds
// heads and splits in a fixed order (in a launch of its own where they are many), so scores are reproducible bit for bit.  Stage B finds the
// k-th largest score (up to 2048 tokens four bits a round with all keys in registers, more of them with a radix select in LDS), keeps
// everything above it plus the first ties in position order, and numbers the survivors in position order; the optional
// gather copies the surviving rows of a [rows, row_elems] matrix.
#include "common.h"
#include "score_plan.h"
#include <algorithm>
#include <type_traits>

using namespace dream;

namespace {

struct ScoreArgs {
    const void *q, *k;
    const int32_t *q_pos;
    float *lse2;   // [ns1, B, Hq, n_q_pad]  log2-domain log-sum-exp of each row over the keys of split s (-inf: none)
    const float *lse_in;   // nullable [B, Hq, n_q]: the caller's natural-log log-sum-exp of every row (pass 1 is skipped)
    float *part;   // [B, Hq, ns2, vis_len]  column sums per head and row split
    int32_t n_q, n_q_pad, n_keys, n_q_heads, n_kv_heads, vis_start, vis_len;
    float *ent_part;    // [ns1, B, Hq, n_q_pad]  expected score of the row under its attention weights, per split (entropy only)
    float *row_entropy, *block_sum;   // entropy of unsplit blocks: nullable [B, Hq, n_q], and [B, Hq, blocks, 2] sums of 32 rows each (else null: entropy_rows_kernel)
    int32_t ns1, ns2;   // most splits of the streamed axis a block has: keys in pass 1, query rows in pass 2
    int64_t lse_split_stride;   // B * Hq * n_q_pad
    int64_t s_max;
    float scale, scale_log2;
    SplitMap map;       // of the pass that is launched
    UnitOrder order;    // (last: what every workgroup reads lies together)
};

// This workgroup's unit and sequence (score_grid() says which index is which).  All arguments that the first loads need are asked for at once, the entry of an order behind them: one after the
// other, each under a condition that the one before decides, they were up to ten trips to memory, as the arguments of a launch are in no cache.  The arguments of one pass, 428 bytes, where
// those of both were 720.  Calls, us, before / now / with the entry asked for beside the others: column sums of one sequence, 4 heads of 128 x 1500 rows 15.6 / 15.4 / 15.5, 8 of 256 x 1500
// 19.1 / 18.2 / 18.5, 32 of 128 x 1280 20.0 / 19.8 / 20.5; both passes, 32 of 128 x 1280 31.8 / 31.7 / 32.5, 4 sequences of 500 24.8 / 24.2 / 25.0; entropy, 32 of 64 x 1600 17.6 / 17.1 / 17.3.
__device__ __forceinline__ SplitUnit own_unit(const ScoreArgs &a, int &b)
{
    SplitMap map = a.map;
    int ordered = a.order.n;
    asm volatile("" : "+s"(map.count[0]), "+s"(map.count[1]), "+s"(map.count[2]), "+s"(map.count[3]), "+s"(map.count[4]), "+s"(map.count[5]), "+s"(map.count[6]), "+s"(map.count[7]), "+s"(ordered)
                 : "s"(a.q), "s"(a.k), "s"(a.q_pos), "s"(a.n_q), "s"(a.n_keys), "s"(a.n_q_heads), "s"(a.n_kv_heads), "s"(a.vis_start), "s"(a.vis_len), "s"(a.s_max));
    b = ordered ? blockIdx.y : blockIdx.z;
    if (ordered)
        return split_unit(map, true, a.order.pair[blockIdx.z >> 1], blockIdx.z);
    return split_unit(map, false, 0, blockIdx.y);
}

// ---- what the two passes share: a stream of 64-row steps from memory straight into LDS ------------------------------------
// Both passes hold one operand of q k^T in registers and stream the other.  Ablations of the first versions (rows through
// registers into padded LDS, 4 waves that each read every row) showed no single bound: at 16 SmolVLM sequences the column-sum
// pass lost 9-25 % when any one of loads, LDS reads, MFMA, exponentials or additions was left out, so the waves wait on each
// other's latencies.  Hence: loads that need no registers, no LDS write instructions and next to no address arithmetic, which also
// leaves room for one more workgroup per CU; no bank conflicts; fragments that serve two MFMA tiles per LDS read.
template <int D>
struct StreamGeom {
    static constexpr int ROW = D * 2, CPR = D / 8, RPI = 64 / CPR;         // bytes and 16-byte chunks of a row; rows per load instruction
    static constexpr int STAGE = STEP * ROW, NLD = STEP / RPI / 4;         // bytes of a step; load instructions of a wave per step
    static constexpr int NS = 2;                                           // stages (a third costs resident workgroups: 154 -> 162 us at 16 SmolVLM sequences)
};

// Position of 16-byte chunk i of row r within the row: i ^ swizzle(r).  A load instruction writes 1024 contiguous bytes, so rows
// cannot be padded; permuted like this, the 16 rows of a fragment read sit in 16 different bank groups.
template <int D>
__device__ __forceinline__ int swizzle(int r)
{
    return D == 64 ? (r >> 1) & 7 : r & 15;
}

// DIRECT: the loads go straight to LDS, which needs 16-byte aligned rows.  Tensors that start anywhere else (a slice of a larger buffer) take
// the same way through registers, with the alignment of their elements and the same results.
template <int D, bool DIRECT>
struct RowStream {
    using G = StreamGeom<D>;
    const unsigned char *base;     // row 0
    int64_t row_bytes;             // between rows
    int n_rows, next;              // rows there are; the next step to load
    uint32_t lds0;
    unsigned char *stage0;
    int wave, lane;
    uint32_t at[G::NLD];           // this lane's byte offsets from the step's first row

    __device__ __forceinline__ void init(const void *rows, int64_t bytes_between, int n, int first_step, unsigned char *lds, int wave_, int lane_)
    {
        base = reinterpret_cast<const unsigned char *>(rows);
        row_bytes = bytes_between;
        n_rows = n;
        next = first_step;
        lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char *)lds;
        stage0 = lds;
        wave = wave_;
        lane = lane_;
#pragma unroll
        for (int j = 0; j < G::NLD; j++) {
            const int row = (wave * G::NLD + j) * G::RPI + lane / G::CPR;
            at[j] = (uint32_t)(row * (int)row_bytes + ((lane % G::CPR) ^ swizzle<D>(row)) * 16);
        }
    }
    // rows past the last one re-read it (nobody uses their scores)
    __device__ __forceinline__ void issue(int stage)
    {
        const int row0 = min(next * STEP, n_rows - 1), left = n_rows - 1 - row0;
        next++;
        const unsigned char *from = base + row0 * row_bytes;
        const uint32_t to = stage * G::STAGE + wave * G::NLD * 1024;
        if (left >= STEP - 1) {
#pragma unroll
            for (int j = 0; j < G::NLD; j++)
                load(from, at[j], to + j * 1024);
        } else {
#pragma unroll
            for (int j = 0; j < G::NLD; j++)
                load(from, min(at[j], (uint32_t)(left * (int)row_bytes) + (at[j] & (G::ROW - 1))), to + j * 1024);
        }
    }
    __device__ __forceinline__ void load(const unsigned char *from, uint32_t offset, uint32_t to)
    {
        if (DIRECT) {
            lds_load16(from, offset, lds0 + to);
        } else {
            const uint16_t *e = reinterpret_cast<const uint16_t *>(from + offset);
            s16x8 v;
#pragma unroll
            for (int i = 0; i < 8; i++)
                v[i] = (short)e[i];
            *reinterpret_cast<s16x8 *>(stage0 + to + lane * 16) = v;
        }
    }
};

// Entropy of a row from its log-sum-exp and its expected score, both in log2 units.  Rounding can leave a tiny negative value for a one-hot row; NaN stays.
__device__ __forceinline__ float entropy_of(float lse, float expected)
{
    const float H = 0.6931471805599453f * (lse - expected);
    return H < 0.0f ? 0.0f : H;
}

// Pass 1: log-sum-exp of every causal row.  One workgroup per (64 query rows, head, sequence, key split).  K is streamed (RowStream, one
// barrier per step of 64 keys); the four waves are two row slots x two key halves of a step, each with one MFMA tile of 32 keys by
// 32 rows.  Scores are formed transposed (lane = query column), so a lane keeps a
// private running (max, sum); the row groups of the wave and the two halves are combined once at the end.  With
// several splits each workgroup writes a partial log-sum-exp that pass 2 combines.
// With ENT the kernel also keeps t = sum_j 2^(x_j - m) x_j, so that the expected score sum_j A_j x_j = t / l of
// the row is known and the row's entropy -sum A log A = LSE - sum A_j s_j (Eq. 2, Section 3.2) needs no
// second pass.
// Measured (attention entropy, all its launches): Pixtral prompt of 1279 tokens 28.6 -> 22.2 us, 16 SmolVLM sequences 251 -> 200 us.
// The held rows as whole lines instead of 16-byte pieces of 16 rows per load: 57.8 -> 49.6 us at 32 LLaVA sequences of 320 tokens.
// The reference raised by octaves and a step's fragments requested together: 22.7 -> 21.7 us and 188 -> 185 us for larger prompts, all launches.
// What bounds it there is the issue of instructions.  Where workgroups are many (take_double()) they hold 128 rows: four row slots, and a wave takes both halves of a step.
// One tile of 32x32 in the place of four of 16x16 is half the MFMAs for the same products, one reference and one pair of sums per lane.  Entropy, all launches, with four tiles, blocks of 64 rows in
// their own order and a launch that forms the entropies / now: 16 SmolVLM sequences 175.7 / 166.2, 16 of 32 x 1200 rows at head_dim 128 149.5 / 134.7, one LLaVA prompt 14.4 / 11.2; the pass alone at
// one Pixtral prompt 18.0 / 17.0: there it is the launch that counts.
template <int D, bool ENT, bool DIRECT, int SLOTS>
__global__ __launch_bounds__(256, 2) void scores_lse_bf16_kernel(ScoreArgs a)
{
    using G = StreamGeom<D>;
    constexpr int NKS = D / 16, HALVES = 4 / SLOTS, TILES = 2 / HALVES;      // TILES: halves of a step that a wave takes
    static_assert(SLOTS == 2 || SLOTS == 4, "two row slots by two halves, or four row slots");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[G::NS * G::STAGE];
    __shared__ float s_half[HALVES == 2 ? SLOTS : 1][ENT ? 3 : 2][COLS];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slot = wave & (SLOTS - 1), half = wave / SLOTS;
    const int c = lane & 31, g = lane >> 5;
    // x walks the heads with the KV head fastest: workgroup ids that share a KV head are congruent mod 8
    // (when there are 8 or more KV heads), so its K is fetched into one XCD's L2 only
    // later row blocks see more keys: they come first
    int b;
    const SplitUnit unit = own_unit(a, b);
    const int kvh = blockIdx.x % a.n_kv_heads, h = kvh * (a.n_q_heads / a.n_kv_heads) + blockIdx.x / a.n_kv_heads;
    const int blk = a.map.count[0] - 1 - unit.rank, split = unit.split;
    // Blocks of 128 rows are counted from the last row up, so that with an odd number of 64s the half empty one is the shortest: the rows 0 to 63
    const int from_end = (a.n_q + BLOCK - 1) / BLOCK - 2 * (unit.rank + 1);
    const int row0 = SLOTS == 2 ? blk * BLOCK : max(from_end, 0) * BLOCK, row_end = SLOTS == 4 && from_end < 0 ? min(BLOCK, a.n_q) : a.n_q;
    const int row = row0 + slot * COLS + c;
    const bool valid = row < row_end;
    int pos = valid ? row : -1;
    // keys this workgroup has to see: without explicit positions, up to its last row
    const int key_lim = a.q_pos ? a.n_keys : min(min(row0 + SLOTS * COLS, row_end), a.n_keys);
    const int n_steps_all = (key_lim + STEP - 1) / STEP;
    const int sps = (n_steps_all + unit.n - 1) / unit.n;
    const int s0 = split * sps, n_steps = max(min(sps, n_steps_all - s0), 0);   // steps s0 .. s0 + n_steps - 1
    // the wave's first and last position (rows that do not exist keep nothing, so they do not count)
    int wave_min_pos = row0 + slot * COLS, wave_max_pos = wave_min_pos < row_end ? min(wave_min_pos + COLS, row_end) - 1 : -1;
    if (a.q_pos) {
        if (valid)
            pos = a.q_pos[(int64_t)b * a.n_q + row];
        wave_max_pos = max(pos, -1);
        wave_min_pos = valid ? pos : 0x7fffffff;
        for (int off = 32; off > 0; off >>= 1) {
            wave_max_pos = max(wave_max_pos, __shfl_xor(wave_max_pos, off));
            wave_min_pos = min(wave_min_pos, __shfl_xor(wave_min_pos, off));
        }
        wave_max_pos = __builtin_amdgcn_readfirstlane(wave_max_pos);
        wave_min_pos = __builtin_amdgcn_readfirstlane(wave_min_pos);
    }

    const uint16_t *kb = reinterpret_cast<const uint16_t *>(a.k) + ((int64_t)b * a.n_kv_heads + kvh) * a.s_max * D;
    RowStream<D, DIRECT> keys;
    keys.init(kb, D * 2, a.n_keys, s0, lds, wave, lane);
    auto first_keys = [&] {
        if (n_steps > 0) {
#pragma unroll
            for (int i = 0; i < G::NS - 1; i++)
                keys.issue(i);
        }
    };
    // the rows come the same way, as whole lines, and once for all waves that hold them: 64 of them into the stage that step 1 will take, 128 into both stages
    // before the keys
    RowStream<D, DIRECT> rows;
    rows.init(reinterpret_cast<const uint16_t *>(a.q) + ((int64_t)b * a.n_q * a.n_q_heads + h) * D, (int64_t)a.n_q_heads * D * 2, a.n_q, row0 / STEP, lds, wave, lane);
    if (SLOTS == 2)
        first_keys();
    else
        rows.issue(0);
    rows.issue(1);
    int frag[NKS];                 // byte offsets of this lane's fragments in a half of a stage
#pragma unroll
    for (int ks = 0; ks < NKS; ks++)
        frag[ks] = c * G::ROW + ((ks * 2 + g) ^ swizzle<D>(c)) * 16;
    bf16x8 qf[NKS];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < NKS; ks++)
        qf[ks] = *reinterpret_cast<const bf16x8 *>(lds + (SLOTS == 2 ? G::STAGE : 0) + slot * COLS * G::ROW + frag[ks]);
    if (SLOTS == 4) {
        __syncthreads();                                         // the rows have been read
        first_keys();
    }
    float m = -INFINITY, l = 0.0f, tx = 0.0f;
    for (int i = 0, stage = 0; i < n_steps; i++) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((G::NS - 2) * G::NLD) : "memory");   // this wave's share of step i has landed
        __syncthreads();                                                               // everybody's has, and step i - 1 is no longer read
        keys.issue(stage == 0 ? G::NS - 1 : stage - 1);
        const unsigned char *st = lds + stage * G::STAGE + half * 32 * G::ROW;
        stage = stage == G::NS - 1 ? 0 : stage + 1;
        const int key0 = (s0 + i) * STEP + half * 32;
        // tile t: keys key0 + t * 32 .. + 31
        auto products = [&](int t, f32x16 &acc) {
            acc = f32x16{};
            // Requested together: the waits then fall behind the first products.  At head_dim 256 four at a time, the next four before the products of the last: 16 at once hold the first product up
            // for longer than the two waves of a SIMD have work for.  Entropy, us, 16 / four at a time (four tiles of 16x16 before: the third): 16 heads x 7417 rows 255 / 240 / 235, 8 x 6003 101.5 / 95.7 / 96.8,
            // 28 x 4 x 2013 162 / 153 / 171.
            constexpr int AT_ONCE = D == 256 ? 4 : NKS, GROUPS = NKS / AT_ONCE;
            bf16x8 kf[2][AT_ONCE];
            auto request = [&](int n) {
#pragma unroll
                for (int i = 0; i < AT_ONCE; i++)
                    kf[n & 1][i] = *reinterpret_cast<const bf16x8 *>(st + t * 32 * G::ROW + frag[n * AT_ONCE + i]);
                __builtin_amdgcn_sched_barrier(0);
            };
            request(0);
#pragma unroll
            for (int n = 0; n < GROUPS; n++) {
                if (n + 1 < GROUPS)
                    request(n + 1);
#pragma unroll
                for (int i = 0; i < AT_ONCE; i++)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[n & 1][i], qf[n * AT_ONCE + i], acc, 0, 0, 0);
                if (n + 1 < GROUPS)
                    __builtin_amdgcn_sched_barrier(0);
            }
        };
        // The row's reference m is raised only when a score exceeds it by 8 octaves: powers of two stay below 2^8, and the sums are
        // rescaled a few times per row instead of in every step.  mult: what still multiplies the scores; masked: some are -inf, the mark of a
        // key that the row does not see (a NaN is no mark: it makes the row's sums NaN)
        auto add_scores = [&](const auto &acc, float mx, float mult, auto masked) {
            if (__any(mx > m + 8.0f)) {
                const float m_new = mx > m + 8.0f ? mx : m, alpha = m_new == m ? 1.0f : __builtin_amdgcn_exp2f(m - m_new);   // (0 when the old reference was -inf)
                m = m_new;
                l *= alpha;
                if (ENT)
                    tx *= alpha;
            }
            const float neg_m = m == -INFINITY ? 0.0f : -m;
            float sum = 0.0f, xsum = 0.0f;
#pragma unroll
            for (int t = 0; t < (int)std::extent<std::remove_reference_t<decltype(acc)>>::value; t++)
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const float x = acc[t][e], p = __builtin_amdgcn_exp2f(fmaf(x, mult, neg_m));
                    sum += p;
                    if (ENT)
                        xsum = fmaf(p, decltype(masked)::value ? fmaxf(x, -3.0e38f) : x, xsum);   // (finite, so that times a probability of 0 it is 0)
                }
            l += sum;
            if (ENT)
                tx = fmaf(xsum, mult, tx);
        };
        // the last key of `n` tiles from tile t on is visible to every row of the wave (all but those on the diagonal): no masking,
        // the maximum is taken before scaling and the scale rides in the exponent's fma
        auto open = [&](int t, int n) { return key0 + (t + n) * 32 - 1 <= wave_min_pos && key0 + (t + n) * 32 - 1 < a.n_keys && a.scale_log2 > 0.0f; };
        auto add_open = [&](const auto &acc) {
            float x = -INFINITY;
#pragma unroll
            for (int t = 0; t < (int)std::extent<std::remove_reference_t<decltype(acc)>>::value; t++)
#pragma unroll
                for (int e = 0; e < 16; e++)
                    x = fmaxf(x, acc[t][e]);
            add_scores(acc, x * a.scale_log2, a.scale_log2, std::false_type{});
        };
        if (TILES == 2 && open(0, TILES)) {
            f32x16 acc[TILES];
#pragma unroll
            for (int t = 0; t < TILES; t++)
                products(t, acc[t]);
            add_open(acc);
            continue;
        }
#pragma unroll
        for (int t = 0; t < TILES; t++) {
            if (key0 + t * 32 > wave_max_pos)
                continue;   // causal: nothing in this tile is visible to this wave's rows
            f32x16 acc[1];
            products(t, acc[0]);
            if (open(t, 1)) {
                add_open(acc);
            } else {
                const int lim = min(pos, a.n_keys - 1) - key0 - t * 32 - g * 4;      // key g * 4 + 8 * (e / 4) + e % 4 is visible up to here
                float mx = -INFINITY;
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const float x = (e >> 2) * 8 + (e & 3) <= lim ? acc[0][e] * a.scale_log2 : -INFINITY;
                    acc[0][e] = x;
                    mx = fmaxf(mx, x);
                }
                add_scores(acc, mx, 1.0f, std::true_type{});
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the loads past the last step have landed before the LDS is given up
    // the two row groups of the wave, then the halves of the steps where two waves took them
    float mt = fmaxf(m, __shfl_xor(m, 32));
    const float wgt = __builtin_amdgcn_exp2f(m - ((mt == -INFINITY) ? 0.0f : mt));
    l *= wgt;
    l += __shfl_xor(l, 32);
    if (ENT) {
        tx *= wgt;
        tx += __shfl_xor(tx, 32);
    }
    m = mt;
    float lw = l, ew = tx;
    if constexpr (HALVES == 2) {
        if (half == 1 && g == 0) {
            s_half[slot][0][c] = m;
            s_half[slot][1][c] = l;
            if (ENT)
                s_half[slot][ENT ? 2 : 1][c] = tx;
        }
        __syncthreads();
        if (half == 1 || g != 0)
            return;
        const float mo = s_half[slot][0][c];
        mt = fmaxf(m, mo);
        const float ms = (mt == -INFINITY) ? 0.0f : mt;
        const float w0 = __builtin_amdgcn_exp2f(m - ms), w1 = __builtin_amdgcn_exp2f(mo - ms);
        lw = l * w0 + s_half[slot][1][c] * w1;
        if (ENT)
            ew = tx * w0 + s_half[slot][ENT ? 2 : 1][c] * w1;
    } else if (g != 0) {
        return;
    }
    const bool some = ENT ? lw != 0.0f : lw > 0.0f;          // (a row with a NaN score: its entropy is NaN, its column sums leave it out)
    const float lse = some ? mt + log2f(lw) : -INFINITY;
    const float expected = ENT && some ? ew / lw : 0.0f;
    if (ENT && a.block_sum) {
        float H = valid && some ? entropy_of(lse, expected) : 0.0f;
        if (valid && a.row_entropy)
            a.row_entropy[((int64_t)b * a.n_q_heads + h) * a.n_q + row] = H;
        for (int off = 16; off > 0; off >>= 1)
            H += __shfl_xor(H, off);
        if (c == 0)
            a.block_sum[(((int64_t)b * a.n_q_heads + h) * a.map.count[0] + blk) * SLOTS + slot] = H;
        return;
    }
    if (valid) {
        const int64_t o = split * a.lse_split_stride + ((int64_t)b * a.n_q_heads + h) * a.n_q_pad + row;
        a.lse2[o] = lse;
        if (ENT)
            a.ent_part[o] = expected;
        if (split == 0)                                      // splits that other blocks have and this one does not: both values, since
            for (int s = unit.n; s < a.ns1; s++) {           // a weight of 0 does not make a NaN left in the workspace harmless
                a.lse2[o + s * a.lse_split_stride] = -INFINITY;
                if (ENT)
                    a.ent_part[o + s * a.lse_split_stride] = 0.0f;
            }
    }
}

// Entropy of every row from pass 1's per-split (log-sum-exp, expected score) pairs (Eq. 2).  One thread per
// (head, row), its pairs requested together; each workgroup also leaves the sum of its 256 entropies for entropy_mean_kernel, which adds the
// workgroup sums of a sequence in a fixed order, so the mean is reproducible.  (The last workgroup to arrive in the place of the second launch: 3 us
// slower at 200 workgroups, for what a release and an acquire between the XCDs' L2s cost.)
// log2_domain: bf16 path (scores in log2 units); otherwise natural units and a single split.
template <int NS1>
__global__ __launch_bounds__(256) void entropy_rows_kernel(ScoreArgs a, int log2_domain, float *row_entropy, float *block_sum)
{
    __shared__ float s_part[4];
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_rows = a.n_q_heads * a.n_q;
    const int i = blockIdx.x * 256 + tid;
    float H = 0.0f;
    if (i < n_rows) {
        const int h = i / a.n_q, r = i - h * a.n_q;
        const int64_t o = ((int64_t)b * a.n_q_heads + h) * a.n_q_pad + r;
        if (log2_domain) {
            float L[NS1], E[NS1];
#pragma unroll
            for (int s = 0; s < NS1; s++) {
                L[s] = a.lse2[s * a.lse_split_stride + o];
                E[s] = a.ent_part[s * a.lse_split_stride + o];
            }
            float M = -INFINITY;
            bool some = false;
#pragma unroll
            for (int s = 0; s < NS1; s++) {
                M = fmaxf(M, L[s]);
                some |= L[s] != -INFINITY;                    // (a NaN, which the maximum drops and the weights below keep)
            }
            if (some) {
                float W = 0.0f, U = 0.0f;
#pragma unroll
                for (int s = 0; s < NS1; s++) {
                    const float w = __builtin_amdgcn_exp2f(L[s] - M);
                    W += w;
                    U += w * E[s];
                }
                H = entropy_of(M + log2f(W), U / W);
            }
        } else {
            const float L = a.lse2[o];
            H = L == INFINITY ? 0.0f : L - a.ent_part[o];
            H = H < 0.0f ? 0.0f : H;
        }
        if (row_entropy)
            row_entropy[((int64_t)b * a.n_q_heads + h) * a.n_q + r] = H;
    }
    float acc = H;
    for (int off = 32; off > 0; off >>= 1)
        acc += __shfl_xor(acc, off);
    if (lane == 0)
        s_part[wave] = acc;
    __syncthreads();
    if (tid == 0)
        block_sum[(int64_t)b * gridDim.x + blockIdx.x] = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
}

// One workgroup per sequence; thread i adds the sums i, i + 256, ... in order, then a fixed tree over lanes and waves.  (One thread adding
// them one after the other took 7.7 us for 160 sums.)  Eight sums are asked for at once, without a condition, since a load under a condition is waited for where the condition
// ends.  The call, us, one after the other / at once: 1280 sums 18.9 / 18.0, 1664 17.9 / 16.4, 4 sequences of 1664 51.2 / 50.1, 4032 91.4 / 90.0.
__global__ __launch_bounds__(256) void entropy_mean_kernel(const float *block_sum, int n_blocks, int n_rows, float *ae)
{
    __shared__ float s_part[4];
    const int b = blockIdx.x, tid = threadIdx.x;
    float t = 0.0f;
    for (int i0 = tid; i0 < n_blocks; i0 += 8 * 256) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; k++)
            v[k] = block_sum[(int64_t)b * n_blocks + min(i0 + k * 256, n_blocks - 1)];
#pragma unroll
        for (int k = 0; k < 8; k++)
            t += i0 + k * 256 < n_blocks ? v[k] : 0.0f;
    }
    for (int off = 32; off > 0; off >>= 1)
        t += __shfl_xor(t, off);
    if ((tid & 63) == 0)
        s_part[tid >> 6] = t;
    __syncthreads();
    if (tid == 0)
        ae[b] = ((s_part[0] + s_part[1]) + (s_part[2] + s_part[3])) / (float)n_rows;
}

// Pass 2: column sums of the probabilities.  One workgroup per (64 visual keys, head, sequence, row split).  The query
// rows are streamed (RowStream); the four waves are two key slots x two row halves of a step, each with the K fragments of 32
// keys in registers.  A lane sums its key columns over the rows it holds; the four row groups and the two halves are
// combined at the end, so every (head, row split, key) sum has one fixed order.  The rows' log-sum-exps (combined from pass
// 1's partial values) and positions are put into LDS for 512 rows at a time.
// Measured (compression with the caller's log-sum-exps, all its launches): LLaVA 25.4 -> 19, Pixtral 37.4 -> 27.1, 16 SmolVLM sequences
// 197 -> 151 us.  What bounds it there is the issue of vector instructions: the counters of that launch (123 us alone) show the vector ALU
// busy 69 % of the time, the matrix cores 25 %, LDS 21 % without a bank conflict, 4.9 waves per SIMD.  Tiles of 32x32, which pass 1 takes, need more
// registers or more LDS reads here and were 3-6 % slower.  Where workgroups are many (take_double()) they hold 128 keys in four key slots, and a wave takes both halves of a
// step: 16 Pixtral sequences of 1279 tokens 148.7 -> 129.7, 32 Gemma3 of 2000 272 -> 243, 16 SmolVLM of 1600 128.4 -> 125.6 us, the same bits.  (8 waves that hold 128 keys, halves
// apart: 3 % at most.)
template <int D, int NS1, bool DIRECT, int SLOTS>
__global__ __launch_bounds__(256, 2) void scores_colsum_bf16_kernel(ScoreArgs a)
{
    using G = StreamGeom<D>;
    constexpr int NKS = D / 32, WINDOW = 512, CT = COLS / 16, HALVES = 4 / SLOTS, TILES = 2 / HALVES;   // TILES: halves of a step that a wave takes
    // At head_dim 256 a SIMD has two waves, which do not cover what the compiler leaves to be waited for: there the log-sum-exps are read before the products and the fragments ahead of theirs.
    // Column sums, us, as at the other head_dims / so: 16 heads x 7000 rows 124 / 121.5, 32 x 4024 123 / 118, 9 sequences of 8 x 2584 127 / 123.5, 8 of 16 x 1280 76.4 / 73.6, one of 8 x 1500 18.8 / 17.7.
    // At head_dim 128 it is the other way: 16 of 32 x 1279 131 / 133.
    constexpr bool FEW_WAVES = D == 256;
    static_assert(SLOTS == 2 || SLOTS == 4, "two key slots by two halves, or four key slots");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[G::NS * G::STAGE];
    __shared__ __attribute__((aligned(16))) float lds_lse[WINDOW];
    __shared__ __attribute__((aligned(16))) int32_t lds_pos[WINDOW];
    __shared__ float s_half[HALVES == 2 ? SLOTS : 1][CT][16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slot = wave & (SLOTS - 1), half = wave / SLOTS;
    const int c = lane & 15, g = lane >> 4;
    const int vis_end = a.vis_start + a.vis_len;
    // x walks the heads with the KV head fastest (see pass 1): the query rows of a head stay in one XCD's L2
    int b;
    const SplitUnit unit = own_unit(a, b);        // earlier key blocks are seen by more rows: they come first
    const int kvh = blockIdx.x % a.n_kv_heads, h = kvh * (a.n_q_heads / a.n_kv_heads) + blockIdx.x / a.n_kv_heads;
    const int blk0 = a.vis_start + unit.rank * (SLOTS * COLS), split = unit.split;
    const int j0 = blk0 + slot * 16 * CT;                 // this wave's keys: j0 + q * 16 + c
    bool kvalid[CT];
#pragma unroll
    for (int q = 0; q < CT; q++) {
        const int key = j0 + q * 16 + c;
        kvalid[q] = key < vis_end && key < a.n_keys;
    }
    // row steps: without explicit positions row r sits at position r, so rows below the block's first key see nothing
    const int n_steps_all = (a.n_q + STEP - 1) / STEP;
    const int s_begin = a.q_pos ? 0 : min(blk0 / STEP, n_steps_all);
    const int sps = (n_steps_all - s_begin + unit.n - 1) / unit.n;
    const int s_first = s_begin + split * sps, n_steps = max(min(sps, n_steps_all - s_first), 0);
    const uint16_t *qb = reinterpret_cast<const uint16_t *>(a.q) + ((int64_t)b * a.n_q * a.n_q_heads + h) * D;
    const float *lrow = a.lse2 + ((int64_t)b * a.n_q_heads + h) * a.n_q_pad;
    RowStream<D, DIRECT> rows;
    rows.init(qb, (int64_t)a.n_q_heads * D * 2, a.n_q, s_first, lds, wave, lane);
    auto first_rows = [&] {
        if (n_steps > 0) {
#pragma unroll
            for (int i = 0; i < G::NS - 1; i++)
                rows.issue(i);
        }
    };
    // the keys come the same way, as whole lines, and once for all waves that hold them: 64 of them into the stage that step 1 will take, 128 into both stages
    // before the rows
    RowStream<D, DIRECT> keys;
    keys.init(reinterpret_cast<const uint16_t *>(a.k) + (((int64_t)b * a.n_kv_heads + kvh) * a.s_max + blk0) * D, D * 2, a.n_keys - blk0, 0, lds, wave, lane);
    if (SLOTS == 2)
        first_rows();
    else
        keys.issue(0);
    keys.issue(1);
    // log-sum-exps over all keys (in log2 units) and positions of rows row0 .. row0 + WINDOW - 1
    auto fill_window = [&](int row0) {
        for (int w = tid; w < min(WINDOW, n_steps * STEP); w += 256) {
            const int r = row0 + w;
            float L = -INFINITY;
            if (r < a.n_q) {
                if (a.lse_in) {
                    L = a.lse_in[((int64_t)b * a.n_q_heads + h) * a.n_q + r] * 1.4426950408889634f;
                } else {
                    float lr[NS1];
#pragma unroll
                    for (int s = 0; s < NS1; s++)
                        lr[s] = lrow[s * a.lse_split_stride + r];
                    L = lr[0];                                   // a single split is taken as it is
                    if (NS1 > 1) {
#pragma unroll
                        for (int s = 1; s < NS1; s++)
                            L = fmaxf(L, lr[s]);
                        float sum = 0.0f;
#pragma unroll
                        for (int s = 0; s < NS1; s++)
                            sum += __builtin_amdgcn_exp2f(lr[s] - (L == -INFINITY ? 0.0f : L));
                        L += log2f(sum);
                    }
                }
                if (a.q_pos)
                    lds_pos[w] = a.q_pos[(int64_t)b * a.n_q + r];
            } else if (a.q_pos) {
                lds_pos[w] = -1;
            }
            lds_lse[w] = L > -INFINITY ? L : INFINITY;           // +inf makes the probability zero: rows that do not exist or see no key
        }
    };
    float cs[TILES][CT];
#pragma unroll
    for (int t = 0; t < TILES; t++)
#pragma unroll
        for (int q = 0; q < CT; q++)
            cs[t][q] = 0.0f;
    int frag[NKS];                 // byte offsets of this lane's fragments in a half of a stage
#pragma unroll
    for (int ks = 0; ks < NKS; ks++)
        frag[ks] = c * G::ROW + ((ks * 4 + g) ^ swizzle<D>(c)) * 16;
    bf16x8 kf[CT][NKS];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int q = 0; q < CT; q++)
#pragma unroll
        for (int ks = 0; ks < NKS; ks++)
            kf[q][ks] = *reinterpret_cast<const bf16x8 *>(lds + (SLOTS == 2 ? G::STAGE : 0) + (slot * CT + q) * 16 * G::ROW + frag[ks]);
    if (SLOTS == 4) {
        __syncthreads();                                         // the keys have been read
        first_rows();
    }
    const bool none = SLOTS == 4 && j0 >= vis_end;               // a wave past the last key only loads
    for (int i = 0, stage = 0; i < n_steps; i++) {
        if (i % (WINDOW / STEP) == 0) {
            if (i > 0)
                __syncthreads();                                 // the last window's steps have been read
            fill_window((s_first + i) * STEP);
        }
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((G::NS - 2) * G::NLD) : "memory");   // this wave's share of step i has landed
        __syncthreads();                                                               // everybody's has, and step i - 1 is no longer read
        rows.issue(stage == 0 ? G::NS - 1 : stage - 1);
        const unsigned char *st = lds + stage * G::STAGE + half * 32 * G::ROW;
        stage = stage == G::NS - 1 ? 0 : stage + 1;
        const int r0 = (s_first + i) * STEP + half * 32, w0 = i % (WINDOW / STEP) * STEP + half * 32;
        // tile t: rows r0 + t * 32 .. + 31, in two accumulators of 16
        auto products = [&](int t, f32x4 (&acc)[CT][2]) {
#pragma unroll
            for (int q = 0; q < CT; q++)
                acc[q][0] = acc[q][1] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (FEW_WAVES) {
                // two key steps at a time, the next two requested before the products of the last: see FEW_WAVES
                constexpr int AT_ONCE = 2, GROUPS = NKS / AT_ONCE;
                bf16x8 f[2][AT_ONCE][2];
                auto request = [&](int n) {
#pragma unroll
                    for (int i = 0; i < AT_ONCE; i++)
#pragma unroll
                        for (int r = 0; r < 2; r++)
                            f[n & 1][i][r] = *reinterpret_cast<const bf16x8 *>(st + (t * 32 + r * 16) * G::ROW + frag[n * AT_ONCE + i]);
                    __builtin_amdgcn_sched_barrier(0);
                };
                request(0);
#pragma unroll
                for (int n = 0; n < GROUPS; n++) {
                    if (n + 1 < GROUPS)
                        request(n + 1);
#pragma unroll
                    for (int i = 0; i < AT_ONCE; i++)
#pragma unroll
                        for (int q = 0; q < CT; q++)
#pragma unroll
                            for (int r = 0; r < 2; r++)
                                acc[q][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[n & 1][i][r], kf[q][n * AT_ONCE + i], acc[q][r], 0, 0, 0);
                    if (n + 1 < GROUPS)
                        __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int ks = 0; ks < NKS; ks++) {
                    const bf16x8 q0 = *reinterpret_cast<const bf16x8 *>(st + t * 32 * G::ROW + frag[ks]);
                    const bf16x8 q1 = *reinterpret_cast<const bf16x8 *>(st + (t * 32 + 16) * G::ROW + frag[ks]);
#pragma unroll
                    for (int q = 0; q < CT; q++) {
                        acc[q][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q0, kf[q][ks], acc[q][0], 0, 0, 0);
                        acc[q][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q1, kf[q][ks], acc[q][1], 0, 0, 0);
                    }
                }
            }
        };
        // the log-sum-exps of the lane's rows of a tile
        auto row_lse = [&](int t, f32x4 (&L)[2]) {
            L[0] = *reinterpret_cast<const f32x4 *>(&lds_lse[w0 + t * 32 + g * 4]);
            L[1] = *reinterpret_cast<const f32x4 *>(&lds_lse[w0 + t * 32 + 16 + g * 4]);
        };
        // every row of the tile sits at or after every key of this wave: nothing to mask
        auto add_open = [&](int t, const f32x4 (&acc)[CT][2], const f32x4 (&L)[2]) {
#pragma unroll
            for (int q = 0; q < CT; q++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    cs[t][q] += __builtin_amdgcn_exp2f(fmaf(acc[q][0][r], a.scale_log2, -L[0][r]));
                    cs[t][q] += __builtin_amdgcn_exp2f(fmaf(acc[q][1][r], a.scale_log2, -L[1][r]));
                }
        };
        if (none)
            continue;
        if (TILES == 2 && !a.q_pos && r0 >= j0 + 16 * CT - 1) {
            f32x4 acc[TILES][CT][2], L[TILES][2];
#pragma unroll
            for (int t = 0; t < TILES; t++) {
                if (FEW_WAVES)
                    row_lse(t, L[t]);
                products(t, acc[t]);
            }
#pragma unroll
            for (int t = 0; t < TILES; t++) {
                if (!FEW_WAVES)
                    row_lse(t, L[t]);
                add_open(t, acc[t], L[t]);
            }
            continue;
        }
#pragma unroll
        for (int t = 0; t < TILES; t++) {
            const int rt = r0 + t * 32;
            if (!a.q_pos && rt + 31 < j0)
                continue;   // causal: these rows sit before this wave's keys
            f32x4 acc[CT][2], L[2];
            if (FEW_WAVES)
                row_lse(t, L);
            products(t, acc);
            if (!FEW_WAVES)
                row_lse(t, L);
            if (!a.q_pos && rt >= j0 + 16 * CT - 1) {
                add_open(t, acc, L);
                continue;
            }
            i32x4 at0 = {0, 1, 2, 3}, at1 = {16, 17, 18, 19};      // positions, or without them the rows from the lane's first one on
            if (a.q_pos) {
                at0 = *reinterpret_cast<const i32x4 *>(&lds_pos[w0 + t * 32 + g * 4]);
                at1 = *reinterpret_cast<const i32x4 *>(&lds_pos[w0 + t * 32 + 16 + g * 4]);
            }
#pragma unroll
            for (int q = 0; q < CT; q++) {
                // rows of the tile from here on see the key: row r of this lane at position at0[r] or at1[r]
                const int key = j0 + q * 16 + c - (a.q_pos ? 0 : rt + g * 4);
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const float p0 = __builtin_amdgcn_exp2f(acc[q][0][r] * a.scale_log2 - L[0][r]);
                    const float p1 = __builtin_amdgcn_exp2f(acc[q][1][r] * a.scale_log2 - L[1][r]);
                    cs[t][q] += key <= at0[r] ? p0 : 0.0f;
                    cs[t][q] += key <= at1[r] ? p1 : 0.0f;
                }
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the loads past the last step have landed before the LDS is given up
#pragma unroll
    for (int q = 0; q < CT; q++) {
#pragma unroll
        for (int t = 0; t < TILES; t++) {
            cs[t][q] += __shfl_xor(cs[t][q], 16);
            cs[t][q] += __shfl_xor(cs[t][q], 32);
        }
        if (HALVES == 2 && half == 1 && g == 0)
            s_half[slot][q][c] = cs[0][q];
    }
    if (HALVES == 2)
        __syncthreads();
    if (half == 1 || g != 0)
        return;
#pragma unroll
    for (int q = 0; q < CT; q++) {
        const int key = j0 + q * 16 + c;
        if (key < vis_end) {
            float *to = a.part + ((int64_t)b * a.n_q_heads + h) * a.ns2 * a.vis_len + (key - a.vis_start);
            to[split * a.vis_len] = kvalid[q] ? cs[0][q] + (HALVES == 2 ? s_half[HALVES == 2 ? slot : 0][q][c] : cs[TILES - 1][q]) : 0.0f;
            if (split == 0)                                  // splits that other blocks have and this one does not
                for (int s = unit.n; s < a.ns2; s++)
                    to[s * a.vis_len] = 0.0f;
        }
    }
}

// ---- float32 tensors: plain vector-ALU versions of the two passes -------------------------------
__global__ __launch_bounds__(256) void scores_lse_f32_kernel(ScoreArgs a, int D)
{
    __shared__ float sq[256];
    __shared__ float red_m[4], red_l[4], red_t[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int kvh = h / (a.n_q_heads / a.n_kv_heads);
    const int pos = a.q_pos ? a.q_pos[(int64_t)b * a.n_q + row] : row;
    const float *q = reinterpret_cast<const float *>(a.q) + (((int64_t)b * a.n_q + row) * a.n_q_heads + h) * D;
    const float *kb = reinterpret_cast<const float *>(a.k) + ((int64_t)b * a.n_kv_heads + kvh) * a.s_max * D;
    if (tid < D)
        sq[tid] = q[tid];
    __syncthreads();
    float m = -INFINITY, l = 0.0f, tx = 0.0f;   // tx = sum_j exp(x_j - m) x_j (used for the entropy only)
    const int lim = min(pos + 1, a.n_keys);
    for (int key = tid; key < lim; key += 256) {
        const float *kr = kb + (int64_t)key * D;
        float dot = 0.0f;
        for (int d = 0; d < D; d++)
            dot += sq[d] * kr[d];
        float x = dot * a.scale;
        float mn = fmaxf(m, x);
        const float al = expf(m - mn), p = expf(x - mn);
        l = l * al + p;
        tx = tx * al + p * x;
        m = mn;
    }
    for (int off = 32; off > 0; off >>= 1) {
        float om = __shfl_xor(m, off), ol = __shfl_xor(l, off), ot = __shfl_xor(tx, off);
        float mn = fmaxf(m, om);
        float ms = (mn == -INFINITY) ? 0.0f : mn;
        l = l * expf(m - ms) + ol * expf(om - ms);
        tx = tx * expf(m - ms) + ot * expf(om - ms);
        m = mn;
    }
    if (lane == 0) {
        red_m[wave] = m;
        red_l[wave] = l;
        red_t[wave] = tx;
    }
    __syncthreads();
    if (tid == 0) {
        float mm = fmaxf(fmaxf(red_m[0], red_m[1]), fmaxf(red_m[2], red_m[3]));
        float ms = (mm == -INFINITY) ? 0.0f : mm;
        float ll = 0.0f, tt = 0.0f;
        for (int w = 0; w < 4; w++) {
            ll += red_l[w] * expf(red_m[w] - ms);
            tt += red_t[w] * expf(red_m[w] - ms);
        }
        const int64_t o = ((int64_t)b * a.n_q_heads + h) * a.n_q_pad + row;
        const bool some = a.ent_part ? ll != 0.0f : ll > 0.0f;   // (as in the bf16 kernel)
        a.lse2[o] = some ? mm + logf(ll) : INFINITY;             // natural log here
        if (a.ent_part)
            a.ent_part[o] = some ? tt / ll : 0.0f;
    }
}

__global__ __launch_bounds__(64) void scores_colsum_f32_kernel(ScoreArgs a, int D)
{
    const int j = blockIdx.x * 64 + threadIdx.x, h = blockIdx.y, b = blockIdx.z;
    if (j >= a.vis_len)
        return;
    const int key = a.vis_start + j;
    const int kvh = h / (a.n_q_heads / a.n_kv_heads);
    float cs = 0.0f;
    if (key < a.n_keys) {
        const float *kr = reinterpret_cast<const float *>(a.k) + (((int64_t)b * a.n_kv_heads + kvh) * a.s_max + key) * D;
        const float *lrow = a.lse_in ? a.lse_in + ((int64_t)b * a.n_q_heads + h) * a.n_q : a.lse2 + ((int64_t)b * a.n_q_heads + h) * a.n_q_pad;
        for (int row = 0; row < a.n_q; row++) {
            int pos = a.q_pos ? a.q_pos[(int64_t)b * a.n_q + row] : row;
            if (key > pos || lrow[row] == -INFINITY)   // (a caller's log-sum-exp of a row that sees no key)
                continue;
            const float *q = reinterpret_cast<const float *>(a.q) + (((int64_t)b * a.n_q + row) * a.n_q_heads + h) * D;
            float dot = 0.0f;
            for (int d = 0; d < D; d++)
                dot += q[d] * kr[d];
            cs += expf(dot * a.scale - lrow[row]);
        }
    }
    a.part[((int64_t)b * a.n_q_heads + h) * a.vis_len + j] = cs;
}

// ---- stage B ----------------------------------------------------------------------------------
// One workgroup of 1024 threads per sequence; everything lives in LDS.  Scores are mapped to unsigned keys
// whose order is the order of the floats; the k-th largest key is found by a most-significant-digit radix
// select (4 passes of 256-bin histograms built with integer LDS atomics, so nothing depends on scheduling).
// A token is kept iff its key is above the threshold, or equal to it and among the first `need` such tokens
// in position order (equal scores resolve toward the lower index); survivors are compacted in position order.
// Dynamic LDS: vis_len keys, then 256 histogram bins, 32 wave totals and 4 control words.
__device__ __forceinline__ uint32_t order_key(float x)
{
    x += 0.0f;   // -0 and +0 are equal scores: give them one key
    const uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? max(~u, 1u) : (u | 0x80000000u);   // (never 0, the key of no token: the NaN of all ones would have it)
}

__global__ __launch_bounds__(1024) void topk_keep_kernel(const float *part, int n_heads, const float *scores_in,
                                                         float *scores_out, int vis_start, int vis_len, int k,
                                                         int32_t *kept_idx)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    uint32_t *key = reinterpret_cast<uint32_t *>(smem_raw);
    int32_t *hist = reinterpret_cast<int32_t *>(key + vis_len);
    int32_t *wave_tot = hist + 256;   // [2][16]
    int32_t *ctl = wave_tot + 32;     // [0] chosen bin, [1] remaining need
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int j = tid; j < vis_len; j += 1024) {
        float x;
        if (scores_in) {
            x = scores_in[(int64_t)b * vis_len + j];
        } else {
            x = 0.0f;
            for (int h0 = 0; h0 < n_heads; h0 += 32) {   // up to 32 loads in flight, added in head order
                float t32[32];
#pragma unroll
                for (int i = 0; i < 32; i++)
                    t32[i] = h0 + i < n_heads ? part[((int64_t)b * n_heads + h0 + i) * vis_len + j] : 0.0f;
#pragma unroll
                for (int i = 0; i < 32; i++)
                    x += t32[i];
            }
        }
        if (scores_out)
            scores_out[(int64_t)b * vis_len + j] = x;
        key[j] = order_key(x);
    }
    if (k <= 0)
        return;
    // ---- radix select of the k-th largest key
    uint32_t prefix = 0, mask = 0;
    int need = k;
    for (int shift = 24; shift >= 0; shift -= 8) {
        if (tid < 256)
            hist[tid] = 0;
        __syncthreads();
        for (int j = tid; j < vis_len; j += 1024) {
            const uint32_t u = key[j];
            if ((u & mask) == prefix)
                atomicAdd(&hist[(u >> shift) & 255u], 1);
        }
        __syncthreads();
        if (wave == 0) {
            // lane l owns bins 4l..4l+3; walk down from the top bin until `need` keys are covered
            int c4[4], tot = 0;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                c4[i] = hist[4 * lane + i];
                tot += c4[i];
            }
            // suffix scan over lanes: keys in bins owned by higher lanes
            int incl = tot;
            for (int off = 1; off < 64; off <<= 1) {
                int v = __shfl_down(incl, off);
                if (lane + off < 64)
                    incl += v;
            }
            const int above = incl - tot;
            if (above < need && need <= above + tot) {
                int rem = need - above, bin = 4 * lane + 3;
#pragma unroll
                for (int i = 3; i >= 0; i--) {
                    if (rem > 0) {
                        bin = 4 * lane + i;
                        if (rem <= c4[i]) {
                            ctl[0] = bin;
                            ctl[1] = rem;
                            rem = 0;
                        } else {
                            rem -= c4[i];
                        }
                    }
                }
            }
        }
        __syncthreads();
        prefix |= (uint32_t)ctl[0] << shift;
        mask |= 255u << shift;
        need = ctl[1];
        __syncthreads();
    }
    const uint32_t tau = prefix;   // key of the k-th largest; `need` of the keys equal to it are kept
    // ---- ordered compaction: thread t owns the contiguous slice [t*per, (t+1)*per)
    const int per = (vis_len + 1023) / 1024;
    const int lo = min(tid * per, vis_len), hi = min(lo + per, vis_len);
    int gt = 0, eq = 0;
    for (int j = lo; j < hi; j++) {
        const uint32_t u = key[j];
        gt += u > tau;
        eq += u == tau;
    }
    int gi = gt, ei = eq;   // inclusive scans inside the wave
    for (int off = 1; off < 64; off <<= 1) {
        int a = __shfl_up(gi, off), c = __shfl_up(ei, off);
        if (lane >= off) {
            gi += a;
            ei += c;
        }
    }
    if (lane == 63) {
        wave_tot[wave] = gi;
        wave_tot[16 + wave] = ei;
    }
    __syncthreads();
    int g_before = gi - gt, e_before = ei - eq;
    for (int w = 0; w < wave; w++) {
        g_before += wave_tot[w];
        e_before += wave_tot[16 + w];
    }
    int out = g_before + min(e_before, need);
    for (int j = lo; j < hi; j++) {
        const uint32_t u = key[j];
        bool keep = u > tau;
        if (u == tau) {
            keep = e_before < need;
            e_before++;
        }
        if (keep)
            kept_idx[(int64_t)b * k + out++] = vis_start + j;
    }
}

// Adds the partial column sums of 64 tokens of one sequence, all heads and row splits, into row 0: one workgroup of 16 waves, wave w the
// rows w, w + 16, ... in order, then the waves in order.  (The sums are a few hundred KB: one CU pulls them in about 5 us, the
// many of this launch at once.)
__global__ __launch_bounds__(1024) void sum_parts_kernel(float *part, int n_parts, int vis_len)
{
    __shared__ float s_sum[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = blockIdx.x * 64 + lane;
    float *at = part + (int64_t)blockIdx.y * n_parts * vis_len + min(j, vis_len - 1);
    float x = 0.0f;
    for (int i0 = wave; i0 < n_parts; i0 += 16 * 8) {
        float t[8];
#pragma unroll
        for (int u = 0; u < 8; u++)
            t[u] = i0 + 16 * u < n_parts ? at[(int64_t)(i0 + 16 * u) * vis_len] : 0.0f;
#pragma unroll
        for (int u = 0; u < 8; u++)
            x += t[u];
    }
    s_sum[wave][lane] = x;
    __syncthreads();
    if (wave == 0 && j < vis_len) {
        x = s_sum[0][lane];
#pragma unroll
        for (int w = 1; w < 16; w++)
            x += s_sum[w][lane];
        *at = x;
    }
}

// Sums over lanes by register moves (shuffles are trips through LDS, and here one waits for the other): over the four rows of 16 lanes, and over the lower 32 lanes.
__device__ __forceinline__ int sum_across_rows(int n)
{
    const auto a = __builtin_amdgcn_permlane16_swap((uint32_t)n, (uint32_t)n, false, false);
    n = (int)(a[0] + a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap((uint32_t)n, (uint32_t)n, false, false);
    return (int)(b[0] + b[1]);
}
template <int ROT>
__device__ __forceinline__ uint32_t row_rotate_bits(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + ROT, 0xf, 0xf, false);
}
__device__ __forceinline__ int sum_of_32(int n)
{
    n += (int)row_rotate_bits<8>(n);
    n += (int)row_rotate_bits<4>(n);
    n += (int)row_rotate_bits<2>(n);
    n += (int)row_rotate_bits<1>(n);
    return __builtin_amdgcn_readlane(n, 0) + __builtin_amdgcn_readlane(n, 16);
}
// The bits that all values of a row of 16 lanes have, and those that any has.
__device__ __forceinline__ void row_bits(uint32_t &all, uint32_t &any)
{
    all &= row_rotate_bits<8>(all); any |= row_rotate_bits<8>(any);
    all &= row_rotate_bits<4>(all); any |= row_rotate_bits<4>(any);
    all &= row_rotate_bits<2>(all); any |= row_rotate_bits<2>(any);
    all &= row_rotate_bits<1>(all); any |= row_rotate_bits<1>(any);
}

// Up to 2048 visual tokens: the same selection, and the copy of the kept rows where it is asked for.  NR: tokens per lane if one wave held
// them all.  Latency bound, so it is built from few dependent steps.  The k-th largest key is found four bits a round: lane
// (trial, group) of wave w counts the keys at or above one of 16 trial values in a quarter of the wave's sixteenth of the tokens
// (16 lanes read the same four keys at once), and the search ends as soon as a value keeps exactly k; survivors are numbered
// with ballots.  The search starts with the first four bits in which keys differ, and what is counted is summed by register moves: LLaVA 22.0 -> 21.5 us the whole call, with the
// log-sum-exps given two Gemma3 prompts 17.9 -> 16.2, two SmolVLM prompts 29.8 -> 27.7, 16 132.5 -> 130.7.  Several
// workgroups per sequence all find the same selection and copy some of the kept rows each, which is faster than a launch for the copy.
// n_parts partial sums a token are added here (a thread takes VEC tokens and every n_groups-th partial row, the groups meet in LDS in
// order) where they are few; of a sum formed by sum_parts_kernel n_parts is 1 and the rows of a sequence are `stride` apart.
// Measured, LLaVA prompt (576 tokens, 128 partial rows) / 16 SmolVLM prompts (1088 tokens, 32), us: one kernel for sums and selection and a gather
// 9.8 + 3.3 / 18.5 + 7.7; here sums 3.0, selection with gather 6.2 / sums 4.8, selection 9.8, gather 7.5.
struct GatherArgs {
    const unsigned char *src;      // NULL: no gather
    unsigned char *dst;
    int64_t n_rows_src, row_bytes;
    int32_t lanes;                 // threads per row (a power of two)
};
template <int NR>
__global__ __launch_bounds__(1024) void select_kernel(const float *part, int64_t stride, int n_parts, const float *scores_in, float *scores_out, int vis_start,
                                                      int vis_len, int k, int vec, int32_t *kept_idx, GatherArgs ga)
{
    constexpr int V = NR * 64;
    __shared__ __attribute__((aligned(16))) float s_sum[4096 > V ? 4096 : V];   // [group][vis_len]; then the kept tokens
    __shared__ __attribute__((aligned(16))) uint32_t s_key[V];
    __shared__ int s_cnt[2][16][16];
    __shared__ int s_chunk[32];
    __shared__ uint32_t s_bits[2][16];
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float *mine = scores_in ? scores_in + (int64_t)b * vis_len : part + b * stride;
    const bool many = !scores_in && n_parts > 1;
    int n_groups = 1;
    if (many) {
        const int cols = vec ? vis_len / 4 : vis_len;                   // (vec: rows of partial sums are 16-byte aligned)
        n_groups = min(max(1024 / cols, 1), min(n_parts, 4096 / vis_len));
        for (int col = tid % cols, grp = tid / cols; grp < n_groups && col < cols; col += vec ? cols : 1024) {
            if (vec) {
                const f32x4 *src = reinterpret_cast<const f32x4 *>(mine + (int64_t)grp * vis_len) + col;
                const int64_t step = (int64_t)n_groups * (vis_len / 4);
                f32x4 x = {0.f, 0.f, 0.f, 0.f};
                for (int i = grp; i < n_parts; i += n_groups * 16) {
                    f32x4 t[16];
#pragma unroll
                    for (int u = 0; u < 16; u++)
                        t[u] = i + u * n_groups < n_parts ? src[u * step] : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int u = 0; u < 16; u++)
                        x += t[u];
                    src += 16 * step;
                }
                reinterpret_cast<f32x4 *>(s_sum + grp * vis_len)[col] = x;
            } else {
                const float *src = mine + (int64_t)grp * vis_len + col;
                float x = 0.0f;
#pragma unroll 8
                for (int i = grp; i < n_parts; i += n_groups)
                    x += src[(int64_t)(i - grp) * vis_len];
                s_sum[grp * vis_len + col] = x;
            }
        }
        __syncthreads();
    }
    uint32_t all = ~0u, any = 0u;                                        // bits that all keys, any key of this thread's have
    for (int j = tid; j < V; j += 1024) {
        uint32_t key = 0u;                                               // below every score's key
        if (j < vis_len) {
            float x = 0.0f;
            if (!many) {
                x = mine[j];
            } else {
                for (int g = 0; g < n_groups; g++)
                    x += s_sum[g * vis_len + j];
            }
            if (scores_out && blockIdx.x == 0)
                scores_out[(int64_t)b * vis_len + j] = x;
            key = order_key(x);
            all &= key;
            any |= key;
        }
        s_key[j] = key;
    }
    if (k <= 0)
        return;
    row_bits(all, any);
    all = ((uint32_t)__builtin_amdgcn_readlane(all, 0) & (uint32_t)__builtin_amdgcn_readlane(all, 16)) & ((uint32_t)__builtin_amdgcn_readlane(all, 32) & (uint32_t)__builtin_amdgcn_readlane(all, 48));
    any = ((uint32_t)__builtin_amdgcn_readlane(any, 0) | (uint32_t)__builtin_amdgcn_readlane(any, 16)) | ((uint32_t)__builtin_amdgcn_readlane(any, 32) | (uint32_t)__builtin_amdgcn_readlane(any, 48));
    if (lane == 0) {
        s_bits[0][wave] = all;
        s_bits[1][wave] = any;
    }
    __syncthreads();
    all = s_bits[0][lane & 15];
    any = s_bits[1][lane & 15];
    row_bits(all, any);
    u32x4 key[NR / 4];
    const int group = lane >> 4;
#pragma unroll
    for (int r = 0; r < NR / 4; r++)
        key[r] = reinterpret_cast<const u32x4 *>(s_key)[(wave * 4 + group) * (NR / 4) + r];
    // the largest value with at least k keys at or above it, four bits a round from the first in which keys differ
    const uint32_t common = __builtin_amdgcn_readfirstlane(all), differ = __builtin_amdgcn_readfirstlane(any & ~all);
    const int top = differ ? (31 - __builtin_clz(differ)) & ~3 : -4;
    uint32_t tau = top < 0 ? common : common & ~0u << top << 4;
    int at_tau = vis_len;
    for (int shift = top; shift >= 0 && at_tau != k; shift -= 4) {
        const uint32_t trial = max(tau | ((uint32_t)(lane & 15) << shift), 1u);    // (key 0 is no token)
        int n = 0;
#pragma unroll
        for (int r = 0; r < NR / 4; r++)
#pragma unroll
            for (int e = 0; e < 4; e++)
                n += key[r][e] >= trial ? 1 : 0;
        n = sum_across_rows(n);
        auto cnt = s_cnt[(shift >> 2) & 1];
        if (group == 0)
            cnt[wave][lane] = n;
        __syncthreads();
        int c = (cnt[group * 4][lane & 15] + cnt[group * 4 + 1][lane & 15]) + (cnt[group * 4 + 2][lane & 15] + cnt[group * 4 + 3][lane & 15]);
        c = sum_across_rows(c);
        const int digit = 63 - __builtin_clzll(__ballot(c >= k && lane < 16));    // (trial 0 of the digit always has k keys)
        tau |= (uint32_t)digit << shift;
        at_tau = __builtin_amdgcn_readlane(c, digit);
    }
    // how many keys are above it and equal to it before every chunk of 64; with more keys than asked for the first of those equal to it
    // are kept, in position order
    constexpr int CHUNKS = NR;
    for (int ch = wave; ch < CHUNKS; ch += 16) {
        const uint32_t u = s_key[ch * 64 + lane];
        const int gt = __popcll(__ballot(u > tau)), eq = __popcll(__ballot(u == tau && u != 0u));
        if (lane == 0)
            s_chunk[ch] = gt | eq << 16;
    }
    __syncthreads();
    const int counts = lane < CHUNKS ? s_chunk[lane] : 0;                // (at most 2048 of either: the halves do not meet)
    const int need = k - (sum_of_32(counts) & 0xffff);
    int32_t *s_kept = reinterpret_cast<int32_t *>(s_sum);
    for (int ch = wave; ch < CHUNKS; ch += 16) {
        const int before = sum_of_32(lane < ch ? counts : 0), g_before = before & 0xffff, e_before = before >> 16;
        const uint32_t u = s_key[ch * 64 + lane];
        const uint64_t below = (1ull << lane) - 1ull, ties = __ballot(u == tau && u != 0u);
        const bool keep = u > tau || (u == tau && u != 0u && e_before + (int)__popcll(ties & below) < need);
        const uint64_t kept = __ballot(keep);
        if (keep) {
            const int at = g_before + min(e_before, need) + (int)__popcll(kept & below), token = vis_start + ch * 64 + lane;
            if (blockIdx.x == 0)
                kept_idx[(int64_t)b * k + at] = token;
            s_kept[at] = token;
        }
    }
    if (!ga.src)
        return;
    __syncthreads();
    const int lanes = ga.lanes, per = 1024 / lanes, col = tid & (lanes - 1);
    const unsigned char *src = ga.src + (int64_t)b * ga.n_rows_src * ga.row_bytes;
    unsigned char *dst = ga.dst + (int64_t)b * k * ga.row_bytes;
    const bool wide = ((ga.row_bytes | (uintptr_t)src | (uintptr_t)dst) & 15) == 0;
    for (int t = blockIdx.x * per + tid / lanes; t < k; t += gridDim.x * per) {
        const unsigned char *s = src + (int64_t)s_kept[t] * ga.row_bytes;
        unsigned char *d = dst + (int64_t)t * ga.row_bytes;
        if (wide) {
            for (int64_t i = col; i < ga.row_bytes / 16; i += lanes)
                reinterpret_cast<uint4 *>(d)[i] = reinterpret_cast<const uint4 *>(s)[i];
        } else {
            for (int64_t i = col; i < ga.row_bytes; i += lanes)
                d[i] = s[i];
        }
    }
}

__global__ __launch_bounds__(256) void gather_rows_kernel(const unsigned char *src, int64_t n_rows_src, int64_t row_bytes,
                                                          const int32_t *kept_idx, int k, unsigned char *dst)
{
    const int t = blockIdx.x, b = blockIdx.y;
    const int64_t srow = kept_idx[(int64_t)b * k + t];
    const unsigned char *s = src + ((int64_t)b * n_rows_src + srow) * row_bytes;
    unsigned char *d = dst + ((int64_t)b * k + t) * row_bytes;
    if (((row_bytes | (uintptr_t)s | (uintptr_t)d) & 15) == 0) {
        for (int64_t i = threadIdx.x; i < row_bytes / 16; i += 256)
            reinterpret_cast<uint4 *>(d)[i] = reinterpret_cast<const uint4 *>(s)[i];
    } else {
        for (int64_t i = threadIdx.x; i < row_bytes; i += 256)
            d[i] = s[i];
    }
}

template <int D, bool ENT, bool DIRECT>
void launch_lse(bool wide, dim3 grid, hipStream_t st, const ScoreArgs &a)
{
    if constexpr (DIRECT && D != 64)
        if (wide) {
            hipLaunchKernelGGL((scores_lse_bf16_kernel<D, ENT, true, 4>), grid, dim3(256), 0, st, a);
            return;
        }
    hipLaunchKernelGGL((scores_lse_bf16_kernel<D, ENT, DIRECT, 2>), grid, dim3(256), 0, st, a);
}

template <int D, bool DIRECT>
void launch_colsum(int ns1, bool wide, dim3 grid, hipStream_t st, const ScoreArgs &a)
{
    if constexpr (DIRECT)
        if (wide) {
            hipLaunchKernelGGL((scores_colsum_bf16_kernel<D, 1, true, 4>), grid, dim3(256), 0, st, a);
            return;
        }
    switch (ns1) {
    case 1:  hipLaunchKernelGGL((scores_colsum_bf16_kernel<D, 1, DIRECT, 2>), grid, dim3(256), 0, st, a); break;
    case 2:  hipLaunchKernelGGL((scores_colsum_bf16_kernel<D, 2, DIRECT, 2>), grid, dim3(256), 0, st, a); break;
    case 4:  hipLaunchKernelGGL((scores_colsum_bf16_kernel<D, 4, DIRECT, 2>), grid, dim3(256), 0, st, a); break;
    default: hipLaunchKernelGGL((scores_colsum_bf16_kernel<D, 8, DIRECT, 2>), grid, dim3(256), 0, st, a); break;
    }
}

// With an order of the units: unit by unit.  Without: sequence by sequence, so that the heads at work fit the caches.
dim3 score_grid(const dream_attn_desc *desc, int units, const UnitOrder &order)
{
    return order.n ? dim3(desc->n_q_heads, desc->batch, units) : dim3(desc->n_q_heads, units, desc->batch);
}

// whether the rows of q and k start at multiples of 16 bytes (a row is D * 2 bytes, a multiple of 128)
bool rows_aligned(const void *q, const void *k) { return ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k)) & 15) == 0; }

// calls f with the head dimension, and whether the rows of q and k are 16-byte aligned (see RowStream), as compile-time constants
template <class F>
void with_rows(int head_dim, const void *q, const void *k, F f)
{
    auto with_dim = [&](auto direct) {
        if (head_dim == 64)
            f(std::integral_constant<int, 64>{}, direct);
        else if (head_dim == 128)
            f(std::integral_constant<int, 128>{}, direct);
        else
            f(std::integral_constant<int, 256>{}, direct);
    };
    if (rows_aligned(q, k))
        with_dim(std::true_type{});
    else
        with_dim(std::false_type{});
}

// the selection kernel's dynamic LDS holds up to DREAM_MAX_VISUAL scores
int ensure_topk_lds(const char *who)
{
    static std::atomic<uint64_t> done{0};
    return raise_lds_limit(done, reinterpret_cast<const void *>(&topk_keep_kernel), DREAM_MAX_VISUAL * 4 + (256 + 32 + 4) * 4, who);
}

}  // namespace

namespace dream {
int compress_init() { return ensure_topk_lds("dream_init"); }
}  // namespace dream

extern "C" {

size_t dream_visual_compress_workspace(const dream_attn_desc *desc, int32_t n_q, int32_t vis_len)
{
    if (!desc || desc->batch < 1 || desc->n_q_heads < 1 || n_q < 1)
        return DREAM_WORKSPACE_MIN_BYTES;
    return compress_most(desc->batch, desc->n_q_heads, desc->head_dim, n_q, vis_len, desc->dtype);
}

int dream_visual_compress(const dream_attn_desc *desc, const void *q, const int32_t *q_pos, int32_t n_q,
                          const void *k_cache, int32_t n_keys, int32_t vis_start, int32_t vis_len,
                          int32_t keep_num, int32_t keep_den, const float *scores_in, const float *row_lse_in,
                          float *scores_out, int32_t *kept_idx, int32_t *n_kept_host, const void *gather_src, int64_t n_rows_src,
                          void *gather_dst, int64_t row_elems, void *workspace, size_t workspace_bytes, void *stream)
{
    const char *who = "dream_visual_compress";
    if (!desc)
        return fail(DREAM_ERR_INVALID_ARG, "%s: desc is NULL", who);
    if (desc->batch < 1 || desc->batch > 65535)
        return fail(DREAM_ERR_INVALID_ARG, "%s: batch %d outside [1, 65535]", who, desc->batch);
    if (keep_den <= 0 || keep_num < 0 || keep_num > keep_den)
        return fail(DREAM_ERR_INVALID_ARG, "%s: keep ratio %d/%d is not in [0, 1]", who, keep_num, keep_den);
    if (vis_start < 0 || vis_len < 0)
        return fail(DREAM_ERR_INVALID_ARG, "%s: negative visual span", who);
    if (vis_len > DREAM_MAX_VISUAL)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: vis_len %d exceeds %d", who, vis_len, DREAM_MAX_VISUAL);
    if (desc->dtype != DREAM_F32 && desc->dtype != DREAM_BF16)
        return fail(DREAM_ERR_INVALID_ARG, "%s: unknown dtype %d", who, desc->dtype);
    const int k = (int)(((int64_t)vis_len * keep_num + keep_den / 2) / keep_den);
    if (k > 0 && !kept_idx)
        return fail(DREAM_ERR_INVALID_ARG, "%s: kept_idx is NULL", who);
    if ((gather_src == nullptr) != (gather_dst == nullptr))
        return fail(DREAM_ERR_INVALID_ARG, "%s: gather_src and gather_dst must be given together", who);
    if (gather_src && (row_elems < 1 || n_rows_src < (int64_t)vis_start + vis_len))
        return fail(DREAM_ERR_INVALID_ARG, "%s: gather needs row_elems >= 1 and n_rows_src >= vis_start + vis_len", who);
    hipStream_t st = as_stream(stream);
    const float *part = nullptr;
    int n_heads = 0;
    if (!scores_in && vis_len > 0) {
        if (desc->n_q_heads < 1 || desc->n_kv_heads < 1 || desc->n_q_heads % desc->n_kv_heads || desc->n_q_heads > 65535)
            return fail(DREAM_ERR_INVALID_ARG, "%s: bad head counts %d / %d", who, desc->n_q_heads, desc->n_kv_heads);
        if (desc->head_dim != 64 && desc->head_dim != 128 && desc->head_dim != 256)
            return fail(DREAM_ERR_UNSUPPORTED, "%s: head_dim %d not in {64,128,256}", who, desc->head_dim);
        if (!q || !k_cache)
            return fail(DREAM_ERR_INVALID_ARG, "%s: q and k_cache are required when scores_in is NULL", who);
        if (n_q < 1 || n_keys < 1 || n_keys > desc->s_max)
            return fail(DREAM_ERR_INVALID_ARG, "%s: need n_q >= 1 and 1 <= n_keys <= s_max", who);
        if (!q_pos && n_q > n_keys)
            return fail(DREAM_ERR_INVALID_ARG, "%s: %d rows at positions 0..n_q-1 but only %d keys", who, n_q, n_keys);
        if ((int64_t)vis_start + vis_len > n_keys)
            return fail(DREAM_ERR_INVALID_ARG, "%s: visual span [%d, %d) exceeds the %d live keys", who, vis_start, vis_start + vis_len, n_keys);
        const CompressPlan p = compress_plan(desc->batch, desc->n_q_heads, desc->head_dim, n_q, n_keys, vis_start, vis_len, desc->dtype, q_pos != nullptr, false, row_lse_in != nullptr, rows_aligned(q, k_cache));
        const size_t need = compress_most(desc->batch, desc->n_q_heads, desc->head_dim, n_q, vis_len, desc->dtype);
        if (!workspace || workspace_bytes < need)
            return fail(DREAM_ERR_WORKSPACE, "%s: workspace of %zu bytes, %zu needed", who, workspace_bytes, need);
        ScoreArgs a;
        a.q = q; a.k = k_cache; a.q_pos = q_pos;
        a.lse2 = reinterpret_cast<float *>(static_cast<char *>(workspace) + p.off_lse);
        a.part = reinterpret_cast<float *>(static_cast<char *>(workspace) + p.off_part);
        a.n_q = n_q; a.n_q_pad = p.n_q_pad; a.n_keys = n_keys;
        a.ns1 = row_lse_in ? 1 : p.ns1; a.ns2 = p.ns2; a.map = p.map1; a.order = p.order1; a.ent_part = a.row_entropy = a.block_sum = nullptr; a.lse_in = row_lse_in;
        a.lse_split_stride = (int64_t)desc->batch * desc->n_q_heads * p.n_q_pad;
        a.n_q_heads = desc->n_q_heads; a.n_kv_heads = desc->n_kv_heads;
        a.vis_start = vis_start; a.vis_len = vis_len; a.s_max = desc->s_max;
        a.scale = desc->scale != 0.0f ? desc->scale : 1.0f / sqrtf((float)desc->head_dim);
        a.scale_log2 = a.scale * 1.4426950408889634f;
        if (desc->dtype == DREAM_BF16) {
            if (p.units1 > 65535)
                return fail(DREAM_ERR_UNSUPPORTED, "%s: n_q %d too large for the score grids", who, n_q);
            const dim3 g1 = score_grid(desc, p.units1, p.order1);
            const dim3 g2 = score_grid(desc, p.units2, p.order2);
            // pass 1 (the rows' log-sum-exps) only when the caller does not bring them
            with_rows(desc->head_dim, q, k_cache, [&](auto dim, auto direct) {
                constexpr int D = decltype(dim)::value;
                constexpr bool DIRECT = decltype(direct)::value;
                if (!row_lse_in)
                    launch_lse<D, false, DIRECT>(p.wide1, g1, st, a);
                a.map = p.map2;
                a.order = p.order2;
                launch_colsum<D, DIRECT>(a.ns1, p.wide2, g2, st, a);
            });
        } else {
            if (n_q > 65535 * 1)
                return fail(DREAM_ERR_UNSUPPORTED, "%s: too many rows for the float32 path", who);
            if (!row_lse_in) {
                hipLaunchKernelGGL(scores_lse_f32_kernel, dim3(n_q, desc->n_q_heads, desc->batch), dim3(256), 0, st, a, desc->head_dim);
            }
            hipLaunchKernelGGL(scores_colsum_f32_kernel, dim3(ceil_div(vis_len, 64), desc->n_q_heads, desc->batch), dim3(64), 0, st, a, desc->head_dim);
        }
        int rc = check_launch("visual score kernels");
        if (rc)
            return rc;
        part = a.part;
        n_heads = desc->n_q_heads * p.ns2;
    }
    if (n_kept_host)
        *n_kept_host = k;
    const int64_t row_bytes = gather_src ? row_elems * (desc->dtype == DREAM_F32 ? 4 : 2) : 0;
    if (vis_len > 0 && (k > 0 || scores_out)) {
        if (vis_len <= 2048) {
            // From 64 KB of partial sums a sequence on a launch of its own adds them; see sum_parts_kernel.
            int64_t stride = (int64_t)n_heads * vis_len;
            if (part && stride >= 16384) {
                hipLaunchKernelGGL(sum_parts_kernel, dim3(ceil_div(vis_len, 64), desc->batch), dim3(1024), 0, st, const_cast<float *>(part), n_heads, vis_len);
                if (int rc = check_launch("sum_parts_kernel"))
                    return rc;
                n_heads = 1;
            }
            // The selection's own workgroups copy the rows while one round of them does it: each finds the selection for itself, 4.6 us of the
            // 6.2 with 72 workgroups for one LLaVA prompt (4.6 and a gather of 2.7 us apart), but 22 us with 32 workgroups for each of 16 SmolVLM
            // prompts (9.8 and 7.5 us apart).
            GatherArgs ga = {nullptr, static_cast<unsigned char *>(gather_dst), n_rows_src, row_bytes, 1024};
            int wgs = 1;
            if (gather_src && k > 0) {
                while (ga.lanes > 64 && ga.lanes / 2 >= row_bytes / 16)
                    ga.lanes /= 2;
                wgs = ceil_div(k, 1024 / ga.lanes);
                if ((int64_t)wgs * desc->batch <= 256)
                    ga.src = static_cast<const unsigned char *>(gather_src);
                else
                    wgs = 1;
            }
            const int vec = vis_len % 4 == 0 && (reinterpret_cast<uintptr_t>(part) & 15) == 0;
            static constexpr decltype(&select_kernel<4>) SELECT[] = {select_kernel<4>,  select_kernel<8>,  select_kernel<12>, select_kernel<16>,
                                                                     select_kernel<20>, select_kernel<24>, select_kernel<28>, select_kernel<32>};
            hipLaunchKernelGGL(SELECT[(vis_len - 1) / 256], dim3(wgs, desc->batch), dim3(1024), 0, st, part, stride, n_heads, scores_in, scores_out, vis_start,
                               vis_len, k, vec, kept_idx, ga);
            if (ga.src)
                return check_launch("select_kernel");
        } else {
            const size_t lds = (size_t)vis_len * 4 + (256 + 32 + 4) * 4;
            if (int rc = ensure_topk_lds(who))
                return rc;
            hipLaunchKernelGGL(topk_keep_kernel, dim3(desc->batch), dim3(1024), lds, st, part, n_heads, scores_in, scores_out,
                               vis_start, vis_len, k, kept_idx);
        }
        int rc = check_launch("selection kernel");
        if (rc)
            return rc;
    }
    if (gather_src && k > 0) {
        hipLaunchKernelGGL(gather_rows_kernel, dim3(k, desc->batch), dim3(256), 0, st,
                           static_cast<const unsigned char *>(gather_src), n_rows_src, row_bytes, kept_idx, k,
                           static_cast<unsigned char *>(gather_dst));
        return check_launch("gather_rows_kernel");
    }
    return DREAM_OK;
}

size_t dream_attention_entropy_workspace(const dream_attn_desc *desc, int32_t n_q)
{
    if (!desc || desc->batch < 1 || desc->n_q_heads < 1 || n_q < 1)
        return DREAM_WORKSPACE_MIN_BYTES;
    const int64_t heads = (int64_t)desc->n_q_heads * desc->batch;
    const size_t part = align_up(most_splits(ceil_div(n_q, BLOCK), heads, desc->head_dim, desc->dtype) * heads * ((n_q + 15) / 16 * 16) * sizeof(float), 256);
    const size_t sums = align_up((size_t)desc->batch * ceil_div((int64_t)desc->n_q_heads * n_q, 256) * sizeof(float), 256);
    return DREAM_WORKSPACE_MIN_BYTES + 2 * part + sums;
}

int dream_attention_entropy(const dream_attn_desc *desc, const void *q, const int32_t *q_pos, int32_t n_q, const void *k_cache,
                            int32_t n_keys, float *row_entropy, float *ae, void *workspace, size_t workspace_bytes, void *stream)
{
    const char *who = "dream_attention_entropy";
    if (!desc || !q || !k_cache || !ae)
        return fail(DREAM_ERR_INVALID_ARG, "%s: NULL argument", who);
    if (desc->batch < 1 || desc->batch > 65535)
        return fail(DREAM_ERR_INVALID_ARG, "%s: batch %d outside [1, 65535]", who, desc->batch);
    if (desc->dtype != DREAM_F32 && desc->dtype != DREAM_BF16)
        return fail(DREAM_ERR_INVALID_ARG, "%s: unknown dtype %d", who, desc->dtype);
    if (desc->n_q_heads < 1 || desc->n_kv_heads < 1 || desc->n_q_heads % desc->n_kv_heads || desc->n_q_heads > 65535)
        return fail(DREAM_ERR_INVALID_ARG, "%s: bad head counts %d / %d", who, desc->n_q_heads, desc->n_kv_heads);
    if (desc->head_dim != 64 && desc->head_dim != 128 && desc->head_dim != 256)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: head_dim %d not in {64,128,256}", who, desc->head_dim);
    if (n_q < 1 || n_keys < 1 || n_keys > desc->s_max)
        return fail(DREAM_ERR_INVALID_ARG, "%s: need n_q >= 1 and 1 <= n_keys <= s_max", who);
    if (!q_pos && n_q > n_keys)
        return fail(DREAM_ERR_INVALID_ARG, "%s: %d rows at positions 0..n_q-1 but only %d keys", who, n_q, n_keys);
    const CompressPlan p = compress_plan(desc->batch, desc->n_q_heads, desc->head_dim, n_q, n_keys, 0, 0, desc->dtype, q_pos != nullptr, true, false, rows_aligned(q, k_cache));
    const size_t part = align_up((size_t)p.ns1 * desc->batch * desc->n_q_heads * p.n_q_pad * sizeof(float), 256);
    const int n_blocks = ceil_div((int64_t)desc->n_q_heads * n_q, 256);
    const size_t need = dream_attention_entropy_workspace(desc, n_q);
    if (!workspace || workspace_bytes < need)
        return fail(DREAM_ERR_WORKSPACE, "%s: workspace of %zu bytes, %zu needed", who, workspace_bytes, need);
    hipStream_t st = as_stream(stream);
    ScoreArgs a;
    a.q = q; a.k = k_cache; a.q_pos = q_pos;
    // Blocks that are not split leave entropies in the place of partial values, and their sums, two of a block's 64 rows, fit where those would stand.
    const bool whole = desc->dtype == DREAM_BF16 && p.ns1 == 1;
    float *block_sum = reinterpret_cast<float *>(static_cast<char *>(workspace) + DREAM_WORKSPACE_MIN_BYTES + (whole ? 0 : 2 * part));
    a.row_entropy = whole ? row_entropy : nullptr;
    a.block_sum = whole ? block_sum : nullptr;
    a.lse2 = reinterpret_cast<float *>(static_cast<char *>(workspace) + DREAM_WORKSPACE_MIN_BYTES);
    a.lse_in = nullptr;
    a.ent_part = reinterpret_cast<float *>(static_cast<char *>(workspace) + DREAM_WORKSPACE_MIN_BYTES + part);
    a.part = nullptr;
    a.n_q = n_q; a.n_q_pad = p.n_q_pad; a.n_keys = n_keys;
    a.n_q_heads = desc->n_q_heads; a.n_kv_heads = desc->n_kv_heads;
    a.vis_start = 0; a.vis_len = 0; a.s_max = desc->s_max;
    a.ns1 = p.ns1; a.ns2 = 1; a.map = p.map1; a.order = p.order1;
    a.lse_split_stride = (int64_t)desc->batch * desc->n_q_heads * p.n_q_pad;
    a.scale = desc->scale != 0.0f ? desc->scale : 1.0f / sqrtf((float)desc->head_dim);
    a.scale_log2 = a.scale * 1.4426950408889634f;
    if (desc->dtype == DREAM_BF16) {
        if (p.units1 > 65535)
            return fail(DREAM_ERR_UNSUPPORTED, "%s: n_q %d too large for the score grid", who, n_q);
        const dim3 g1 = score_grid(desc, p.units1, p.order1);
        with_rows(desc->head_dim, q, k_cache, [&](auto dim, auto direct) {
            constexpr int D = decltype(dim)::value;
            constexpr bool DIRECT = decltype(direct)::value;
            launch_lse<D, true, DIRECT>(p.wide1, g1, st, a);
        });
    } else {
        if (n_q > 65535)
            return fail(DREAM_ERR_UNSUPPORTED, "%s: too many rows for the float32 path", who);
        hipLaunchKernelGGL(scores_lse_f32_kernel, dim3(n_q, desc->n_q_heads, desc->batch), dim3(256), 0, st, a, desc->head_dim);
    }
    int rc = check_launch("entropy score kernel");
    if (rc)
        return rc;
    if (!whole) {
        static constexpr decltype(&entropy_rows_kernel<1>) ROWS[] = {entropy_rows_kernel<1>, entropy_rows_kernel<2>, entropy_rows_kernel<4>, entropy_rows_kernel<8>};
        hipLaunchKernelGGL(ROWS[p.ns1 == 8 ? 3 : p.ns1 / 2], dim3(n_blocks, desc->batch), dim3(256), 0, st, a, desc->dtype == DREAM_BF16 ? 1 : 0, row_entropy,
                           block_sum);
    }
    hipLaunchKernelGGL(entropy_mean_kernel, dim3(desc->batch), dim3(256), 0, st, block_sum, whole ? desc->n_q_heads * p.map1.count[0] * (p.wide1 ? 4 : 2) : n_blocks,
                       desc->n_q_heads * n_q, ae);
    return check_launch("entropy reduction kernels");
}

}  // extern "C"
