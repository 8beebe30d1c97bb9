// dream_project_rows: the linear maps of Eq. 1 (Section 3.1), Q = E W_Q, K = S W_K, V = S W_V, for the few
// feature rows a decode step adds (the frontier's draft features, the accepted tokens' target features), with
// the result written straight to where attention reads it: head-split rows of a K/V cache
// [B, H, s_max, D] at row_base[b] + row_index[b, r] (cache append), or a dense [B, R, H, D] tensor (queries).
//
// M = B*R is small (<= a few hundred) and the weight matrix [N, hidden] is large, so the call is bound by
// streaming the weights once from HBM.  One workgroup owns 16 output features (16 weight rows, contiguous in
// memory); its 4 waves split the hidden dimension, each computing C^T[n][m] += W[n][k] X[m][k] with
// v_mfma_f32_16x16x32_bf16 (A = weight rows, B = feature rows).  With at most 16 feature rows (the paper's
// shapes) a wave fetches 256 contiguous bytes of each row at a time and passes them through a private LDS area
// to reach the operand layout: nobody else reads those bytes, but an operand-layout load touches 16 rows x 64
// bytes per instruction, half cache lines, and measures 10-13 % slower.  With more rows, and where its eight waves serve fewer rows better (few feature tiles:
// dream_project_rows_multi has the lines), project_rows_kernel (below) is used.  The partial tiles are summed through LDS in wave order and the rows are rounded to bf16 and scattered.
// Roofline: HBM, N*hidden*2 weight bytes per call.  The weights are loaded without the nontemporal hint: the next level
// reads them again, and what the memory-side cache has kept of them by then is worth more than the hint (drafting 6 levels:
// LLaVA 243 -> 237 us, 8 SmolVLM sequences 285 -> 279; a single call on cold weights is 0-3 us faster but for LLaVA at 10
// rows, 19.2 -> 20.6).
#include <type_traits>
#include "common.h"

using namespace dream;

namespace {

constexpr int NWAVE = 4;   // of project_kernel (8 waves of this kernel measured 5-8 % slower on the narrower maps, 2 no faster)

struct ProjJob {
    const uint16_t *x;
    uint16_t *out;
    const int32_t *row_base, *row_index;
    int32_t n_heads;
};

// What stands ahead of the weights' first loads comes as plain arguments, which are in scalar registers when a wave starts (14 dwords of them): the weights of the jobs, the ends of the
// jobs' workgroup ranges (consecutive; the last end where there is no further job) and the sizes.  The rest is a trip to memory, taken while the weights are on their way.
// (With everything in one structure, looked through job by job, a workgroup made four such trips one after the other ahead of its first load, and two behind its last product, for
// row_base and row_index, which are asked for at the start now: us a call of three maps, before / now, weights in the memory-side cache: 1 row SmolVLM 5.2 / 4.4, LLaVA 16.4 / 15.6,
// 20 rows SmolVLM 6.9 / 6.3, Gemma3 11.8 / 11.1, 80 rows SmolVLM 10.1 / 8.5, Pixtral 19.7 / 18.0, LLaVA 28.5 / 25.9; in HBM 80 rows Gemma3 22.2 / 20.4, LLaVA 40.6 / 39.5.)
struct ProjArgs {
    ProjJob job[DREAM_MAX_PROJ_JOBS];
    int32_t n_rows;      // R: rows per sequence
    int32_t head_dim;
    int32_t row_groups;  // project_rows_kernel: workgroups that share the rows of a weight tile
    int64_t s_max;       // cache mode only
};
static_assert(DREAM_MAX_PROJ_JOBS == 4, "the kernels' arguments");
// (m_and_lack: B * R, at most 2^20, and from bit 24 on, 2 bits a job, by how many feature tiles its last workgroup has fewer than the others)
#define PROJ_PARAMS const uint16_t *w0, const uint16_t *w1, const uint16_t *w2, const uint16_t *w3, int end0, int end1, int end2, int end3, int hidden, uint32_t m_and_lack, ProjArgs args
#define PROJ_SELECT(wg) select_job(w0, w1, w2, w3, end0, end1, end2, end3, m_and_lack, wg)

// The job a workgroup belongs to (uniform), its place among that job's, and how many feature tiles fewer it has.
struct ProjView {
    const uint16_t *w;
    int job, at, lack;
};
__device__ __forceinline__ ProjView select_job(const uint16_t *w0, const uint16_t *w1, const uint16_t *w2, const uint16_t *w3, int end0, int end1, int end2, int end3,
                                               uint32_t m_and_lack, int wg)
{
    ProjView a;
    a.job = wg >= end2 ? 3 : wg >= end1 ? 2 : wg >= end0 ? 1 : 0;
    a.w = wg >= end2 ? w3 : wg >= end1 ? w2 : wg >= end0 ? w1 : w0;
    a.at = wg - (wg >= end2 ? end2 : wg >= end1 ? end1 : wg >= end0 ? end0 : 0);
    const int end = wg >= end2 ? end3 : wg >= end1 ? end2 : wg >= end0 ? end1 : end0;
    a.lack = wg + 1 == end ? m_and_lack >> (24 + 2 * a.job) & 3 : 0;
    return a;
}

// The job's arguments, all asked for at once.
__device__ __forceinline__ ProjJob job_arguments(const ProjArgs &args, int j)
{
    const ProjJob job = args.job[j];
    asm volatile("" ::"s"(job.x), "s"(job.out), "s"(job.row_base), "s"(job.row_index), "s"(job.n_heads), "s"(args.n_rows), "s"(args.head_dim),
                 "s"(args.row_groups), "s"(args.s_max));
    return job;
}

// Where feature row m belongs: its sequence, and the two numbers whose sum is the row in that sequence's cache (or among its rows).  Asked for early, added up behind the products.
struct RowPlace {
    int base, index;
};
__device__ __forceinline__ RowPlace ask_row(const ProjJob &job, int m, int n_rows)
{
    const int b = m / n_rows, r = m - b * n_rows;
    RowPlace p = {0, r};
    if (job.row_base) {
        p.base = job.row_base[b];
        if (job.row_index)
            p.index = job.row_index[m];
    }
    return p;
}

// The lane's four results, outputs n0 + g*4 .. +3 of feature row m, which belongs at `row`, to where they belong.
__device__ __forceinline__ void store_row_piece(const ProjArgs &args, const ProjJob &job, int m, int m_total, int row, int n0, int g, f32x4 sum)
{
    const bool cache = job.row_base != nullptr;
    if (m >= m_total || (cache && (row < 0 || row >= args.s_max)))      // a row outside the cache is dropped, never written
        return;
    const int h = n0 / args.head_dim, d0 = n0 % args.head_dim;
    const int b = m / args.n_rows;
    bf16x4 o;
#pragma unroll
    for (int i = 0; i < 4; i++)
        o[i] = (__bf16)sum[i];
    const int64_t at = cache ? ((int64_t)b * job.n_heads + h) * args.s_max + row : (int64_t)m * job.n_heads + h;
    *reinterpret_cast<bf16x4 *>(job.out + at * args.head_dim + d0 + g * 4) = o;
}

// At most 16 feature rows, XJ * 4 of them loaded.  (With XJ a variable every load of a row is under a condition, and the waits count for the worst of them.)
template <int XJ>
__global__ __launch_bounds__(64 * NWAVE) void project_kernel(PROJ_PARAMS)
{
    const ProjView a = PROJ_SELECT(blockIdx.x);
    const int m_total = m_and_lack & 0xffffff;
    __shared__ __attribute__((aligned(16))) float s_part[NWAVE][64][4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int n0 = a.at * 16;
    const int K = hidden, kw = K / NWAVE;          // this wave's slice of the hidden dimension
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    // Rows are fetched 256 contiguous bytes at a time (4 rows per load instruction: full cache lines) into
    // a wave-private LDS area and read back in operand layout; loading the operands directly would make
    // every instruction touch 16 rows x 64 bytes.
    constexpr int SS = 128, RSTR = SS + 8;             // elements of a row per super-step; padded LDS row stride
    constexpr int LPR = SS / 8, RPI = 64 / LPR, NI = 16 / RPI;   // lanes per row, rows per instruction, instructions per 16 rows
    __shared__ __attribute__((aligned(16))) uint16_t s_stage[NWAVE][2][16 * RSTR];
    uint16_t *lw = s_stage[wave][0], *lx = s_stage[wave][1];
    const int lrow = lane / LPR, lcol = (lane % LPR) * 8;
    const int n_ss = (kw + SS - 1) / SS;
    const uint16_t *wsrc = a.w + (int64_t)n0 * K + wave * kw;
    static_assert(XJ <= NI, "rows");
    const uint16_t *xsrc = nullptr;
    auto column = [&](int s) {
        s = min(s, n_ss - 1);                              // the prefetch past the end re-reads and is dropped
        const int nvalid = min(SS, kw - s * SS);
        return s * SS + (lcol < nvalid ? lcol : 0);
    };
    auto issue_w = [&](int col, u32x4 (&wr)[NI]) {
#pragma unroll
        for (int j = 0; j < NI; j++)
            wr[j] = *reinterpret_cast<const u32x4 *>(wsrc + (int64_t)(j * RPI + lrow) * K + col);
    };
    auto issue_x = [&](int col, u32x4 (&xr)[XJ]) {
#pragma unroll
        for (int j = 0; j < XJ; j++) {     // feature rows are fetched RPI at a time, only as many as exist
            const int m = min(j * RPI + lrow, m_total - 1);
            xr[j] = *reinterpret_cast<const u32x4 *>(xsrc + (int64_t)m * K + col);
        }
    };
    // one super-step: registers -> LDS, request the super-step that reuses these registers, multiply
    auto step = [&](int s, u32x4 (&wr)[NI], u32x4 (&xr)[XJ]) {
#pragma unroll
        for (int j = 0; j < NI; j++) {
            *reinterpret_cast<u32x4 *>(lw + (j * RPI + lrow) * RSTR + lcol) = wr[j];
            if (j < XJ)     // (the other LDS rows feed output columns that are never stored)
                *reinterpret_cast<u32x4 *>(lx + (j * RPI + lrow) * RSTR + lcol) = xr[j < XJ ? j : 0];
        }
        issue_w(column(s + 1), wr);
        issue_x(column(s + 1), xr);
        wave_lds_fence();
        // (a wave's share is a multiple of 64: the last step may be half a one)
        auto multiply = [&](auto n) {
            bf16x8 af[n], bfr[n];
#pragma unroll
            for (int ks = 0; ks < n; ks++) {
                af[ks] = *reinterpret_cast<const bf16x8 *>(lw + c * RSTR + ks * 32 + g * 8);
                bfr[ks] = *reinterpret_cast<const bf16x8 *>(lx + c * RSTR + ks * 32 + g * 8);
            }
#pragma unroll
            for (int ks = 0; ks < n; ks++)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ks], bfr[ks], acc, 0, 0, 0);
        };
        if (kw - s * SS >= SS)
            multiply(std::integral_constant<int, SS / 32>());
        else
            multiply(std::integral_constant<int, SS / 64>());
        wave_lds_fence();
    };
    u32x4 wr[NI], xr[XJ];
    issue_w(column(0), wr);
    __builtin_amdgcn_sched_barrier(0);                     // (the first weights do not wait for the other arguments)
    const ProjJob job = job_arguments(args, a.job);
    xsrc = job.x + wave * kw;
    issue_x(column(0), xr);
    const RowPlace place = ask_row(job, min(c, m_total - 1), args.n_rows);
    for (int s = 0; s < n_ss; s++)
        step(s, wr, xr);
    // sum the waves' partial tiles in wave order
    *reinterpret_cast<f32x4 *>(s_part[wave][lane]) = acc;
    __syncthreads();
    if (wave == 0) {
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NWAVE; w++)
            sum += *reinterpret_cast<const f32x4 *>(s_part[w][lane]);
        store_row_piece(args, job, c, m_total, place.base + place.index, n0, g, sum);
    }
}

// More than 16 feature rows, or few feature tiles.  Every workgroup reads all of the rows (from L2) beside its own weight rows, so what bounds the
// call is feature rows + weight rows per workgroup times workgroups per CU (a CU pulls 60 to 75 GB/s): a workgroup owns NT tiles of 16 output
// features and MT tiles of 16 rows (up to 128 rows per pass), and the launch picks NT for the fewest bytes through the
// busiest CU.  The hidden dimension is dealt to the 8 waves in steps of 64 elements, 1024 contiguous bytes of every row for the eight;
// each wave passes its 128-byte pieces through LDS that only it uses, the next step's loads in flight meanwhile, and keeps all MT x NT
// tiles: no barrier before the partial tiles meet, and every byte is read from LDS once.  (One wave per row tile, stages shared by the
// workgroup and a barrier per step read the weights once per row tile and left 5 of 8 waves multiplying at 80 rows.  Two steps ahead
// were slower at short hidden dimensions and no faster at long ones.)
// Measured per call of three maps (Q, K, V), shared stages / here: 80 rows SmolVLM 11.4 / 10.3 us, LLaVA 40.9 / 40.0, Pixtral 27.1 / 27.3, 40 rows
// 9.1 / 7.2, 30.4 / 28.4, 21.0 / 20.3 with the weights in HBM; as much of them as the memory-side cache kept from the level before, 80 rows LLaVA
// 34.7 / 28.1, Pixtral 21.9 / 19.1, 20 rows LLaVA 25.3 / 18.0.  Whole drafts of 6 levels are 4 to 12 % faster, the expansion's share included.
// Which calls of up to 16 rows take this one: see dream_project_rows_multi.
constexpr int RW = 8;                                // waves per workgroup
constexpr int MAX_MT = 8;                            // row tiles of a pass
constexpr int STEP = 64, STEP_BYTES = STEP * 2;      // elements, bytes of a row per step
constexpr int TILE_BYTES = 16 * STEP_BYTES;

template <int MT, int NT>
struct RowsGeom {
    static constexpr int STAGE = (MT + NT) * TILE_BYTES;                          // of a wave
    static constexpr int ROWS_OFF = RW * MT * NT * 1024;                           // where the rows belong, behind the partial tiles, which reuse the stages
    static constexpr size_t LDS_BYTES = RW * STAGE > ROWS_OFF + 16 * MT * 4 ? RW * STAGE : ROWS_OFF + 16 * MT * 4;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

template <int MT, int NT>
__global__ __launch_bounds__(64 * RW) void project_rows_kernel(PROJ_PARAMS)
{
    using G = RowsGeom<MT, NT>;
    // one row group: a line of workgroups; several: 8 tiles x groups x eighths of the tiles, so that the workgroups of a weight tile have ids congruent
    // mod 8 (same XCD) and few lie between them
    const int tile = blockIdx.z * 8 + blockIdx.x, group = blockIdx.y;
    if (tile >= end3)
        return;
    const ProjView a = PROJ_SELECT(tile);
    const int m_total = m_and_lack & 0xffffff;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int n_here = NT - a.lack, nt0 = a.at * NT;         // feature tiles of this workgroup
    const int K = hidden, n_steps = (K / STEP - wave + RW - 1) / RW;   // this wave's: steps wave, wave + RW, ...
    unsigned char *stage = smem + wave * G::STAGE;
    // The workgroups of an XCD start at different steps: the rows are a power of two or nearly so apart, so one step's pieces
    // of all rows sit in few L2 channels, and everybody would ask the same ones at the same time (LLaVA, 20 rows: 29 us without, 18 with).
    const int first = n_steps > 0 ? (tile >> 3) % n_steps : 0;
    const int lrow = lane >> 3, lchunk = lane & 7;           // a load instruction: 8 rows x 128 bytes
    const uint16_t *wsrc[NT], *xsrc[MT * 2];
#pragma unroll
    for (int nt = 0; nt < NT; nt++)                          // (tiles past the last repeat it, never stored)
        wsrc[nt] = a.w + ((int64_t)(nt0 + min(nt, n_here - 1)) * 16 + lrow) * K + wave * STEP + lchunk * 8;
    u32x4 wr[NT * 2], xr[MT * 2];
    auto column = [&](int s) {
        const int at = s + first;
        return (at < n_steps ? at : at - n_steps) * (RW * STEP);
    };
    auto load_w = [&](int j, int col) { wr[j] = *reinterpret_cast<const u32x4 *>(wsrc[j / 2] + (j % 2 ? (int64_t)8 * K : 0) + col); };
    auto issue_w = [&](int col) {
#pragma unroll
        for (int j = 0; j < NT * 2; j++)
            load_w(j, col);
    };
    if (n_steps > 0)
        issue_w(column(0));
    __builtin_amdgcn_sched_barrier(0);                       // (the first weights do not wait for the other arguments)
    const ProjJob job = job_arguments(args, a.job);
    int m0 = group * 16 * MT, xj = 0;
    RowPlace place = {0, 0};
    auto load_x = [&](int j, int col) {
        if (j < MT * 2 - 2 || j == 0 || j < xj)              // all but the last tile are full
            xr[j] = *reinterpret_cast<const u32x4 *>(xsrc[j] + col);
    };
    auto issue_x = [&](int col) {
#pragma unroll
        for (int j = 0; j < MT * 2; j++)
            load_x(j, col);
    };
    auto start_rows = [&] {                                  // the pass over the rows from m0 on
        xj = min((m_total - m0 + 7) / 8, MT * 2);
#pragma unroll
        for (int j = 0; j < MT * 2; j++)
            xsrc[j] = job.x + (int64_t)min(m0 + j * 8 + lrow, m_total - 1) * K + wave * STEP + lchunk * 8;
        // Where the rows belong is asked for behind their first pieces; ahead of them with eight row tiles, whose many loads it would wait for.  (Behind, calls of 113 to 128 rows of up to 128 feature tiles,
        // weights in the caches, were up to 2.9 % slower than with the places asked for behind the products, ahead 1.4 %; 128 rows in the mean 0.98 and 0.97 of that time, 33 rows 0.94 and 0.95.)
        constexpr bool PLACES_FIRST = MT == MAX_MT;
        auto ask_places = [&] {
            if (tid < 16 * MT)
                place = ask_row(job, min(m0 + tid, m_total - 1), args.n_rows);
        };
        if (PLACES_FIRST)
            ask_places();
        if (n_steps > 0)
            issue_x(column(0));
        if (!PLACES_FIRST)
            ask_places();
        __builtin_amdgcn_sched_barrier(0);
    };
    start_rows();
    for (;;) {
        f32x4 acc[MT][NT];
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
#pragma unroll
            for (int nt = 0; nt < NT; nt++)
                acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        // chunk p of row r of a tile lies at p ^ (r & 7): the 16 rows of a fragment read sit in different banks
        const int put = lrow * STEP_BYTES + ((lchunk ^ lrow) * 16);
        auto step = [&](int s, bool more) {
            // With 8 row tiles a register is asked for again as soon as its piece is in LDS: writing all 20 KB first left the loads idle (128 rows,
            // weights in HBM, LLaVA 50.2 us, 48.2 so; SmolVLM 15.9 and 15.2; but with one or two steps a wave, hidden dimension 768, 6.6 and 6.9)
            constexpr bool EARLY = MT == 8;
            const int col = more ? column(s + 1) : 0;
#pragma unroll
            for (int j = 0; j < NT * 2; j++) {
                *reinterpret_cast<u32x4 *>(stage + j * 1024 + put) = wr[j];
                if (EARLY && more)
                    load_w(j, col);
            }
#pragma unroll
            for (int j = 0; j < MT * 2; j++) {
                if (j < MT * 2 - 2 || j == 0 || j < xj)
                    *reinterpret_cast<u32x4 *>(stage + (NT * 2 + j) * 1024 + put) = xr[j];
                if (EARLY && more)
                    load_x(j, col);
            }
            if (!EARLY && more) {
                issue_w(col);
                issue_x(col);
            }
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < STEP / 32; i++) {
                const int pos = c * STEP_BYTES + (((i * 4 + g) ^ (c & 7)) * 16);
                bf16x8 wf[NT];
#pragma unroll
                for (int nt = 0; nt < NT; nt++)
                    wf[nt] = *reinterpret_cast<const bf16x8 *>(stage + nt * TILE_BYTES + pos);
#pragma unroll
                for (int mt = 0; mt < MT; mt++) {
                    const bf16x8 xf = *reinterpret_cast<const bf16x8 *>(stage + (NT + mt) * TILE_BYTES + pos);
#pragma unroll
                    for (int nt = 0; nt < NT; nt++)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[nt], xf, acc[mt][nt], 0, 0, 0);
                }
            }
            wave_lds_fence();
        };
        if (n_steps > 0) {                                    // (a wave of a narrow map may have none)
            for (int s = 0; s + 1 < n_steps; s++)
                step(s, true);
            step(n_steps - 1, false);
        }
        // the waves' partial tiles, summed in wave order
        __syncthreads();
        f32x4 *part = reinterpret_cast<f32x4 *>(smem);
        int *s_row = reinterpret_cast<int *>(smem + G::ROWS_OFF);
        if (tid < 16 * MT)
            s_row[tid] = place.base + place.index;
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
#pragma unroll
            for (int nt = 0; nt < NT; nt++)
                part[((mt * NT + nt) * RW + wave) * 64 + lane] = acc[mt][nt];
        __syncthreads();
        for (int t = wave; t < MT * NT; t += RW) {
            f32x4 sum = part[t * RW * 64 + lane];
#pragma unroll
            for (int w = 1; w < RW; w++)
                sum += part[(t * RW + w) * 64 + lane];
            const int mt = t / NT, nt = t - mt * NT;
            if (nt < n_here)
                store_row_piece(args, job, m0 + mt * 16 + c, m_total, s_row[mt * 16 + c], (nt0 + nt) * 16, g, sum);
        }
        m0 += args.row_groups * 16 * MT;
        if (m0 >= m_total)
            return;
        __syncthreads();
        if (n_steps > 0)
            issue_w(column(0));
        start_rows();
    }
}

constexpr int MAX_NT = 3;
constexpr int max_nt(int mt) { return mt == 1 || mt > 6 ? 2 : 3; }   // (what LDS holds; what a call with one row tile takes)

template <int MT, int NT>
int ensure_rows_lds(const char *who)
{
    static std::atomic<uint64_t> done{0};
    return raise_lds_limit(done, reinterpret_cast<const void *>(&project_rows_kernel<MT, NT>), RowsGeom<MT, NT>::LDS_BYTES, who);
}

struct Launch {          // the plain arguments
    const uint16_t *w[DREAM_MAX_PROJ_JOBS];
    int end[DREAM_MAX_PROJ_JOBS];
    int hidden;
    uint32_t m_and_lack;
};

template <int MT, int NT>
int launch_rows(int wgs, hipStream_t st, const Launch &l, const ProjArgs &a)
{
    if (int rc = ensure_rows_lds<MT, NT>("dream_project_rows"))
        return rc;
    const dim3 grid = a.row_groups == 1 ? dim3(wgs) : dim3(8, a.row_groups, ceil_div(wgs, 8));
    hipLaunchKernelGGL((project_rows_kernel<MT, NT>), grid, dim3(64 * RW), (RowsGeom<MT, NT>::LDS_BYTES), st, l.w[0], l.w[1], l.w[2], l.w[3], l.end[0], l.end[1],
                       l.end[2], l.end[3], l.hidden, l.m_and_lack, a);
    return check_launch("project_rows_kernel");
}

// The variants, by row tiles per pass and feature tiles per workgroup: project_init walks the table, a call picks from it.
struct RowsVariant {
    int (*launch)(int, hipStream_t, const Launch &, const ProjArgs &);
    int (*ensure)(const char *);
};
#define ROWS_VARIANTS(MT) {{&launch_rows<MT, 1>, &ensure_rows_lds<MT, 1>}, {&launch_rows<MT, 2>, &ensure_rows_lds<MT, 2>}, {&launch_rows<MT, max_nt(MT)>, &ensure_rows_lds<MT, max_nt(MT)>}}
const RowsVariant ROWS[MAX_MT][MAX_NT] = {ROWS_VARIANTS(1), ROWS_VARIANTS(2), ROWS_VARIANTS(3), ROWS_VARIANTS(4), ROWS_VARIANTS(5),
                                              ROWS_VARIANTS(6), ROWS_VARIANTS(7), ROWS_VARIANTS(8)};
#undef ROWS_VARIANTS

}  // namespace

namespace dream {
int project_init()
{
    for (const auto &row : ROWS)
        for (const RowsVariant &v : row)
            if (int rc = v.ensure("dream_init"))
                return rc;
    return DREAM_OK;
}
}  // namespace dream

extern "C" {

int dream_project_rows_multi(const dream_attn_desc *desc, const dream_proj_job *jobs, int32_t n_jobs, int32_t n_rows, int32_t hidden,
                             void *stream)
{
    const char *who = "dream_project_rows";
    if (!desc || !jobs)
        return fail(DREAM_ERR_INVALID_ARG, "%s: NULL argument", who);
    if (n_jobs < 1 || n_jobs > DREAM_MAX_PROJ_JOBS)
        return fail(DREAM_ERR_INVALID_ARG, "%s: %d jobs outside [1, %d]", who, n_jobs, DREAM_MAX_PROJ_JOBS);
    if (desc->dtype != DREAM_BF16)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: bf16 tensors only", who);
    if (desc->batch < 1 || n_rows < 1 || (int64_t)desc->batch * n_rows > (1 << 20))
        return fail(DREAM_ERR_INVALID_ARG, "%s: batch and n_rows must be positive, batch * n_rows at most 2^20", who);
    if (desc->head_dim < 16 || desc->head_dim % 16)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: head_dim %d is not a positive multiple of 16", who, desc->head_dim);
    if (hidden < 256 || hidden % 256)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: hidden %d is not a positive multiple of 256", who, hidden);
    ProjArgs a = {};
    Launch l = {};
    int64_t tiles = 0;
    for (int j = 0; j < n_jobs; j++) {
        const dream_proj_job &jb = jobs[j];
        if (!jb.x || !jb.w || !jb.out)
            return fail(DREAM_ERR_INVALID_ARG, "%s: NULL tensor in job %d", who, j);
        if (jb.n_heads < 1)
            return fail(DREAM_ERR_INVALID_ARG, "%s: n_heads of job %d must be positive", who, j);
        if (jb.row_base && desc->s_max < 1)
            return fail(DREAM_ERR_INVALID_ARG, "%s: cache output needs s_max", who);
        if (!jb.row_base && jb.row_index)
            return fail(DREAM_ERR_INVALID_ARG, "%s: row_index without row_base in job %d", who, j);
        if ((reinterpret_cast<uintptr_t>(jb.x) | reinterpret_cast<uintptr_t>(jb.w) | reinterpret_cast<uintptr_t>(jb.out)) & 15)
            return fail(DREAM_ERR_INVALID_ARG, "%s: x, w and out must be 16-byte aligned", who);
        tiles += (int64_t)jb.n_heads * desc->head_dim / 16;
        if (tiles > (1 << 24))
            return fail(DREAM_ERR_UNSUPPORTED, "%s: more than 2^24 tiles of 16 output features", who);
        a.job[j].x = static_cast<const uint16_t *>(jb.x); l.w[j] = static_cast<const uint16_t *>(jb.w);
        a.job[j].out = static_cast<uint16_t *>(jb.out); a.job[j].row_base = jb.row_base; a.job[j].row_index = jb.row_index;
        a.job[j].n_heads = jb.n_heads; l.end[j] = (int32_t)tiles;
    }
    const int m_total = desc->batch * n_rows;
    for (int j = n_jobs; j < DREAM_MAX_PROJ_JOBS; j++)
        l.end[j] = (int32_t)tiles;
    a.n_rows = n_rows; l.m_and_lack = m_total; l.hidden = hidden; a.head_dim = desc->head_dim;
    a.s_max = desc->s_max;
    hipStream_t st = as_stream(stream);
    // Up to 16 rows: where there are no more feature tiles than CUs, the eight waves of project_rows_kernel, one tile a workgroup; up to twice as many, two tiles, which pull a row once for both,
    // from 9 rows on and from a hidden dimension of 2048 on, where rows count in what is pulled and eight waves have steps enough, but not with rows a multiple of 8 KB apart, whose pieces sit in few channels;
    // else, and above, where workgroups share CUs unevenly, the smaller workgroups of project_kernel.  us, project_kernel / project_rows_kernel, weights in the memory-side cache and in HBM: 10 rows,
    // 8 tiles of hidden dimension 768 4.0 / 3.3 and 4.1 / 3.4, 128 of 3840 5.0 / 4.6 and 6.1 / 5.6, 256 of 4096 5.9 / 5.7 and 7.0 / 6.7;
    // two tiles: 384 of 5120 (Pixtral, three maps) 11.7 / 10.8 and 15.4 / 14.1, 512 of 3840 (Gemma3) 11.5 / 10.8 and 12.7 / 11.9, 384 of 2048 4.9 / 4.7 and 6.1 / 6.0, but
    // 384 of 4096 7.6 / 9.1 and 11.1 / 12.2, 512 of 4096 11.5 / 11.2 and 13.2 / 16.8, 768 of 4096 (LLaVA) 16.2 / 16.4 and 19.6 / 23.6.  Two tiles on the other side of the lines, 257 to 512 tiles of nine hidden
    // dimensions, project_rows_kernel over project_kernel in the mean: hidden 512 and 1024, 10 rows 1.09 and 1.04; from 2048 on, 1 row 1.01 and 1.02, 5 rows 0.98 and 0.99, 10 rows 0.95 and 0.96, 16 rows 0.90 and 0.91
    // (what is left of a loss at 10 rows: 512 of 5120 14.2 / 14.8 and 17.8 / 17.1).
    const int tiles_16 = tiles <= 256 ? 1 : tiles <= 512 && m_total > 8 && hidden >= 2048 && hidden % 4096 ? 2 : 0;
    if (m_total <= 16 && tiles_16 == 0) {
        auto *kernel = m_total > 12 ? &project_kernel<4> : m_total > 8 ? &project_kernel<3> : m_total > 4 ? &project_kernel<2> : &project_kernel<1>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(64 * NWAVE), 0, st, l.w[0], l.w[1], l.w[2], l.w[3], l.end[0], l.end[1], l.end[2], l.end[3], hidden, l.m_and_lack, a);
        return check_launch("project_kernel");
    }
    // Row tiles per pass (1 for up to 16 rows, else 2 to 8), feature tiles per workgroup and how many workgroups share the rows of a feature tile: the fewest bytes
    // through the busiest CU.  Up to 128 rows are one pass; above, a workgroup goes through as few passes as there have to be, of about equal size, or every pass is a workgroup of its
    // own, which leaves fewer CUs idle and reads weights that another pass has brought to L2.  us, one after the other / side by side: LLaVA 256 rows 72.3 / 53.8 (weights in HBM 84.2 / 66.0),
    // 144 rows 50.1 / 40.3, 1000 rows 266 / 205; SmolVLM 192 rows 19.3 / 17.3, 1000 rows 83.8 / 66.6; hidden dimension 768, 1000 rows 32.7 / 16.4.
    const int m_tiles = ceil_div(m_total, 16), passes = ceil_div(m_tiles, MAX_MT);
    int mt = 0, nt = 1;
    int64_t best = 0;
    auto try_split = [&](int m, int n, int groups) {
        int64_t wgs = 0;
        for (int j = 0; j < n_jobs; j++)
            wgs += ceil_div((int64_t)a.job[j].n_heads * a.head_dim / 16, n);
        const bool fits = groups <= 65535 && wgs <= 8 * 65535 && (wgs + 7) / 8 * 8 * groups <= (1 << 22);      // (a grid's extents, its 2^32 threads)
        if (groups > 1)
            wgs = (wgs + 7) / 8 * 8 * groups;
        const int64_t cost = (wgs + 255) / 256 * (groups > 1 ? 16 * (m + n) * 11 : (m_total + 16 * n * passes) * 10);   // (Gemma3, 1000 rows: 8 % fewer, and 5 % slower)
        if (mt == 0 || (cost < best && (groups == 1 || fits))) {
            best = cost;
            mt = m;
            nt = n;
            a.row_groups = groups;
        }
    };
    a.row_groups = 1;
    if (m_total <= 16) {
        mt = 1;
        nt = tiles_16;
    }
    for (int n = 1; mt != 1 && n <= max_nt(ceil_div(m_tiles, passes)); n++)
        try_split(ceil_div(m_tiles, passes), n, 1);
    if (passes > 1)
        for (int m = 2; m <= MAX_MT; m++)
            for (int n = 1; n <= max_nt(m); n++)
                try_split(m, n, ceil_div(m_tiles, m));
    int wgs = 0;
    for (int j = 0; j < DREAM_MAX_PROJ_JOBS; j++) {
        if (j < n_jobs) {
            const int64_t n = (int64_t)a.job[j].n_heads * a.head_dim / 16;
            wgs += ceil_div(n, nt);
            l.m_and_lack |= (uint32_t)(ceil_div(n, nt) * nt - n) << (24 + 2 * j);
        }
        l.end[j] = wgs;
    }
    return ROWS[mt - 1][nt - 1].launch(wgs, st, l, a);
}

int dream_project_rows(const dream_attn_desc *desc, const void *x, int32_t n_rows, int32_t hidden, const void *w, int32_t n_heads,
                       const int32_t *row_base, const int32_t *row_index, void *out, void *stream)
{
    dream_proj_job job = {x, w, n_heads, row_base, row_index, out};
    return dream_project_rows_multi(desc, &job, 1, n_rows, hidden, stream);
}

}  // extern "C"
