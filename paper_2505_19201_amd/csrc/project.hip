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
// bytes per instruction, half cache lines, and measures 10-13 % slower.  With more rows project_rows_kernel (below)
// is used.  The partial tiles are summed through LDS in wave order and the rows are rounded to bf16 and scattered.
// Roofline: HBM, N*hidden*2 weight bytes per call.  The weights are loaded without the nontemporal hint: the next level
// reads them again, and what the memory-side cache has kept of them by then is worth more than the hint (drafting 6 levels:
// LLaVA 243 -> 237 us, 8 SmolVLM sequences 285 -> 279; a single call on cold weights is 0-3 us faster but for LLaVA at 10
// rows, 19.2 -> 20.6).
#include "common.h"

using namespace dream;

namespace {

constexpr int NWAVE = 4;   // (8 waves measured 5-8 % slower on the narrower maps, 2 no faster)

struct ProjJob {
    const uint16_t *x, *w;
    uint16_t *out;
    const int32_t *row_base, *row_index;
    int32_t n_heads;
    int32_t tile_end;    // one past this job's last workgroup (jobs occupy consecutive workgroup ranges)
};

struct ProjArgs {
    ProjJob job[DREAM_MAX_PROJ_JOBS];
    int32_t n_jobs;
    int32_t n_rows;      // R: rows per sequence
    int32_t m_total;     // B * R
    int32_t hidden, head_dim;
    int32_t row_groups;  // project_rows_kernel: workgroups that share the rows of a weight tile
    int64_t s_max;       // cache mode only
};

// The job a workgroup belongs to (uniform: scalar selects) and the first workgroup of that job.
struct ProjView {
    const uint16_t *x, *w;
    uint16_t *out;
    const int32_t *row_base, *row_index;
    int32_t n_heads, n_rows, m_total, hidden, head_dim;
    int64_t s_max;
    int first;
};
__device__ __forceinline__ ProjView select_job(const ProjArgs &args, int wg)
{
    int ji = 0;
    for (int j = 0; j + 1 < args.n_jobs; j++)
        ji += wg >= args.job[j].tile_end;
    ProjView a;
    a.first = 0;
    a.x = args.job[0].x; a.w = args.job[0].w; a.out = args.job[0].out; a.row_base = args.job[0].row_base;
    a.row_index = args.job[0].row_index; a.n_heads = args.job[0].n_heads;
#pragma unroll
    for (int j = 1; j < DREAM_MAX_PROJ_JOBS; j++)
        if (ji == j) {
            a.x = args.job[j].x; a.w = args.job[j].w; a.out = args.job[j].out; a.row_base = args.job[j].row_base;
            a.row_index = args.job[j].row_index; a.n_heads = args.job[j].n_heads;
            a.first = args.job[j - 1].tile_end;
        }
    a.n_rows = args.n_rows; a.m_total = args.m_total; a.hidden = args.hidden; a.head_dim = args.head_dim; a.s_max = args.s_max;
    return a;
}

// The lane's four results, outputs n0 + g*4 .. +3 of feature row m, to where they belong.
__device__ __forceinline__ void store_row_piece(const ProjView &a, int m, int n0, int g, f32x4 sum)
{
    if (m >= a.m_total)
        return;
    const int h = n0 / a.head_dim, d0 = n0 % a.head_dim;
    const int b = m / a.n_rows, r = m - b * a.n_rows;
    bf16x4 o;
#pragma unroll
    for (int i = 0; i < 4; i++)
        o[i] = (__bf16)sum[i];
    int64_t dst;
    if (a.row_base) {
        const int row = a.row_base[b] + (a.row_index ? a.row_index[(int64_t)b * a.n_rows + r] : r);
        dst = row >= 0 && row < a.s_max ? (((int64_t)b * a.n_heads + h) * a.s_max + row) * a.head_dim + d0 + g * 4 : -1;
    } else {
        dst = (((int64_t)b * a.n_rows + r) * a.n_heads + h) * a.head_dim + d0 + g * 4;
    }
    if (dst >= 0)                                        // a row outside the cache is dropped, never written
        *reinterpret_cast<bf16x4 *>(a.out + dst) = o;
}

// At most 16 feature rows.
__global__ __launch_bounds__(64 * NWAVE) void project_kernel(ProjArgs args)
{
    const ProjView a = select_job(args, blockIdx.x);
    __shared__ __attribute__((aligned(16))) float s_part[NWAVE][64][4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int n0 = ((int)blockIdx.x - a.first) * 16;
    const int K = a.hidden, kw = K / NWAVE;          // this wave's slice of the hidden dimension
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
    const uint16_t *xsrc = a.x + wave * kw;
    const int xj = min((a.m_total + RPI - 1) / RPI, NI);
    auto issue = [&](int s, u32x4 (&wr)[NI], u32x4 (&xr)[NI]) {
        s = min(s, n_ss - 1);                              // the prefetch past the end re-reads and is dropped
        const int nvalid = min(SS, kw - s * SS);
        const int col = s * SS + (lcol < nvalid ? lcol : 0);
#pragma unroll
        for (int j = 0; j < NI; j++) {
            wr[j] = *reinterpret_cast<const u32x4 *>(wsrc + (int64_t)(j * RPI + lrow) * K + col);
            if (j < xj) {   // feature rows are fetched RPI at a time, only as many as exist
                const int m = min(j * RPI + lrow, a.m_total - 1);
                xr[j] = *reinterpret_cast<const u32x4 *>(xsrc + (int64_t)m * K + col);
            }
        }
    };
    // one super-step: registers -> LDS, request the super-step that reuses these registers, multiply
    auto step = [&](int s, u32x4 (&wr)[NI], u32x4 (&xr)[NI]) {
#pragma unroll
        for (int j = 0; j < NI; j++) {
            *reinterpret_cast<u32x4 *>(lw + (j * RPI + lrow) * RSTR + lcol) = wr[j];
            if (j < xj)     // (the other LDS rows feed output columns that are never stored)
                *reinterpret_cast<u32x4 *>(lx + (j * RPI + lrow) * RSTR + lcol) = xr[j];
        }
        issue(s + 1, wr, xr);
        wave_lds_fence();
        const int nvalid = min(SS, kw - s * SS);
#pragma unroll
        for (int ks = 0; ks < SS / 32; ks++) {
            if (ks * 32 < nvalid) {
                const bf16x8 af = *reinterpret_cast<const bf16x8 *>(lw + c * RSTR + ks * 32 + g * 8);
                const bf16x8 bfr = *reinterpret_cast<const bf16x8 *>(lx + c * RSTR + ks * 32 + g * 8);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bfr, acc, 0, 0, 0);
            }
        }
        wave_lds_fence();
    };
    u32x4 wr[NI], xr[NI];
    issue(0, wr, xr);
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
        store_row_piece(a, c, n0, g, sum);
    }
}

// More than 16 feature rows.  Every workgroup reads all of them (from L2) beside its own weight rows, so what bounds the
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
// At 10 rows project_kernel and this one are equal within 5 % but for LLaVA (warm 16.5 against 18.0).
constexpr int RW = 8;                                // waves per workgroup
constexpr int STEP = 64, STEP_BYTES = STEP * 2;      // elements, bytes of a row per step
constexpr int TILE_BYTES = 16 * STEP_BYTES;

template <int MT, int NT>
struct RowsGeom {
    static constexpr int STAGE = (MT + NT) * TILE_BYTES;                          // of a wave
    static constexpr size_t LDS_BYTES = RW * (STAGE > MT * NT * 1024 ? STAGE : MT * NT * 1024);   // (the partial tiles reuse the stages)
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

template <int MT, int NT>
__global__ __launch_bounds__(64 * RW) void project_rows_kernel(ProjArgs args)
{
    using G = RowsGeom<MT, NT>;
    // one row group: a line of workgroups; several: 8 tiles x groups x eighths of the tiles, so that the workgroups of a weight tile have ids congruent
    // mod 8 (same XCD) and few lie between them (a tile past the last repeats it and stores nothing)
    const int tile = blockIdx.z * 8 + blockIdx.x, group = blockIdx.y;
    const ProjView a = select_job(args, tile);
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int n_tiles = a.n_heads * a.head_dim / 16, nt0 = (tile - a.first) * NT;
    const int K = a.hidden, n_steps = (K / STEP - wave + RW - 1) / RW;   // this wave's: steps wave, wave + RW, ...
    unsigned char *stage = smem + wave * G::STAGE;
    // The workgroups of an XCD start at different steps: the rows are a power of two or nearly so apart, so one step's pieces
    // of all rows sit in few L2 channels, and everybody would ask the same ones at the same time (LLaVA, 20 rows: 29 us without, 18 with).
    const int first = n_steps > 0 ? (tile >> 3) % n_steps : 0;
    const int lrow = lane >> 3, lchunk = lane & 7;           // a load instruction: 8 rows x 128 bytes
    for (int m0 = group * 16 * MT; m0 < a.m_total; m0 += args.row_groups * 16 * MT) {
        const uint16_t *wsrc[NT], *xsrc[MT * 2];
#pragma unroll
        for (int nt = 0; nt < NT; nt++)                       // (tiles past the last repeat it, never stored)
            wsrc[nt] = a.w + ((int64_t)min(nt0 + nt, n_tiles - 1) * 16 + lrow) * K + wave * STEP + lchunk * 8;
#pragma unroll
        for (int j = 0; j < MT * 2; j++)
            xsrc[j] = a.x + (int64_t)min(m0 + j * 8 + lrow, a.m_total - 1) * K + wave * STEP + lchunk * 8;
        const int xj = min((a.m_total - m0 + 7) / 8, MT * 2);
        u32x4 wr[NT * 2], xr[MT * 2];
        auto column = [&](int s) {
            const int at = s + first;
            return (at < n_steps ? at : at - n_steps) * (RW * STEP);
        };
        auto load_w = [&](int j, int col) { wr[j] = *reinterpret_cast<const u32x4 *>(wsrc[j / 2] + (j % 2 ? (int64_t)8 * K : 0) + col); };
        auto load_x = [&](int j, int col) {
            if (j < MT * 2 - 2 || j < xj)                     // all but the last tile are full
                xr[j] = *reinterpret_cast<const u32x4 *>(xsrc[j] + col);
        };
        auto issue = [&](int s) {
            const int col = column(s);
#pragma unroll
            for (int j = 0; j < NT * 2; j++)
                load_w(j, col);
#pragma unroll
            for (int j = 0; j < MT * 2; j++)
                load_x(j, col);
        };
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
                if (j < MT * 2 - 2 || j < xj)
                    *reinterpret_cast<u32x4 *>(stage + (NT * 2 + j) * 1024 + put) = xr[j];
                if (EARLY && more)
                    load_x(j, col);
            }
            if (!EARLY && more)
                issue(s + 1);
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
            issue(0);
            for (int s = 0; s + 1 < n_steps; s++)
                step(s, true);
            step(n_steps - 1, false);
        }
        // the waves' partial tiles, summed in wave order
        __syncthreads();
        f32x4 *part = reinterpret_cast<f32x4 *>(smem);
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
            if (nt0 + nt < n_tiles)
                store_row_piece(a, m0 + mt * 16 + c, (nt0 + nt) * 16, g, sum);
        }
        __syncthreads();
    }
}

constexpr int MAX_MT = 8, MAX_NT = 3;
constexpr int max_nt(int mt) { return mt < 7 ? 3 : 2; }   // (what LDS holds)

template <int MT, int NT>
int ensure_rows_lds(const char *who)
{
    static std::atomic<uint64_t> done{0};
    return raise_lds_limit(done, reinterpret_cast<const void *>(&project_rows_kernel<MT, NT>), RowsGeom<MT, NT>::LDS_BYTES, who);
}

template <int MT, int NT>
int launch_rows(int wgs, hipStream_t st, const ProjArgs &a)
{
    if (int rc = ensure_rows_lds<MT, NT>("dream_project_rows"))
        return rc;
    const dim3 grid = a.row_groups == 1 ? dim3(wgs) : dim3(8, a.row_groups, ceil_div(wgs, 8));
    hipLaunchKernelGGL((project_rows_kernel<MT, NT>), grid, dim3(64 * RW), (RowsGeom<MT, NT>::LDS_BYTES), st, a);
    return check_launch("project_rows_kernel");
}

// The variants, by row tiles per pass and feature tiles per workgroup: project_init walks the table, a call picks from it.
struct RowsVariant {
    int (*launch)(int, hipStream_t, const ProjArgs &);
    int (*ensure)(const char *);
};
#define ROWS_VARIANTS(MT) {{&launch_rows<MT, 1>, &ensure_rows_lds<MT, 1>}, {&launch_rows<MT, 2>, &ensure_rows_lds<MT, 2>}, {&launch_rows<MT, max_nt(MT)>, &ensure_rows_lds<MT, max_nt(MT)>}}
const RowsVariant ROWS[MAX_MT - 1][MAX_NT] = {ROWS_VARIANTS(2), ROWS_VARIANTS(3), ROWS_VARIANTS(4), ROWS_VARIANTS(5),
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
        a.job[j].x = static_cast<const uint16_t *>(jb.x); a.job[j].w = static_cast<const uint16_t *>(jb.w);
        a.job[j].out = static_cast<uint16_t *>(jb.out); a.job[j].row_base = jb.row_base; a.job[j].row_index = jb.row_index;
        a.job[j].n_heads = jb.n_heads; a.job[j].tile_end = (int32_t)tiles;
    }
    a.n_jobs = n_jobs; a.n_rows = n_rows; a.m_total = desc->batch * n_rows; a.hidden = hidden; a.head_dim = desc->head_dim;
    a.s_max = desc->s_max;
    hipStream_t st = as_stream(stream);
    if (a.m_total <= 16) {
        hipLaunchKernelGGL(project_kernel, dim3((unsigned)tiles), dim3(64 * NWAVE), 0, st, a);
        return check_launch("project_kernel");
    }
    // Row tiles per pass (2 to 8: there are at least 17 rows), feature tiles per workgroup and how many workgroups share the rows of a feature tile: the fewest bytes
    // through the busiest CU.  Up to 128 rows are one pass; above, a workgroup goes through as few passes as there have to be, of about equal size, or every pass is a workgroup of its
    // own, which leaves fewer CUs idle and reads weights that another pass has brought to L2.  us, one after the other / side by side: LLaVA 256 rows 72.3 / 53.8 (weights in HBM 84.2 / 66.0),
    // 144 rows 50.1 / 40.3, 1000 rows 266 / 205; SmolVLM 192 rows 19.3 / 17.3, 1000 rows 83.8 / 66.6; hidden dimension 768, 1000 rows 32.7 / 16.4.
    const int m_tiles = ceil_div(a.m_total, 16), passes = ceil_div(m_tiles, MAX_MT);
    int mt = 0, nt = 1;
    int64_t best = 0;
    auto try_split = [&](int m, int n, int groups) {
        int64_t wgs = 0;
        for (int j = 0; j < n_jobs; j++)
            wgs += ceil_div((int64_t)a.job[j].n_heads * a.head_dim / 16, n);
        const bool fits = groups <= 65535 && wgs <= 8 * 65535 && (wgs + 7) / 8 * 8 * groups <= (1 << 22);      // (a grid's extents, its 2^32 threads)
        if (groups > 1)
            wgs = (wgs + 7) / 8 * 8 * groups;
        const int64_t cost = (wgs + 255) / 256 * (groups > 1 ? 16 * (m + n) * 11 : (a.m_total + 16 * n * passes) * 10);   // (Gemma3, 1000 rows: 8 % fewer, and 5 % slower)
        if (mt == 0 || (cost < best && (groups == 1 || fits))) {
            best = cost;
            mt = m;
            nt = n;
            a.row_groups = groups;
        }
    };
    a.row_groups = 1;
    for (int n = 1; n <= max_nt(ceil_div(m_tiles, passes)); n++)
        try_split(ceil_div(m_tiles, passes), n, 1);
    if (passes > 1)
        for (int m = 2; m <= MAX_MT; m++)
            for (int n = 1; n <= max_nt(m); n++)
                try_split(m, n, ceil_div(m_tiles, m));
    int wgs = 0;
    for (int j = 0; j < n_jobs; j++) {
        wgs += ceil_div((int64_t)a.job[j].n_heads * a.head_dim / 16, nt);
        a.job[j].tile_end = wgs;
    }
    return ROWS[mt - 2][nt - 1].launch(wgs, st, a);
}

int dream_project_rows(const dream_attn_desc *desc, const void *x, int32_t n_rows, int32_t hidden, const void *w, int32_t n_heads,
                       const int32_t *row_base, const int32_t *row_index, void *out, void *stream)
{
    dream_proj_job job = {x, w, n_heads, row_base, row_index, out};
    return dream_project_rows_multi(desc, &job, 1, n_rows, hidden, stream);
}

}  // extern "C"
