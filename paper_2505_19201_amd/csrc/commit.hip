// dream_kv_commit: after verification the K/V rows of the accepted root-to-node path become the next rows of
// the cached prefix and every other tree row is dropped (Section 2.1: everything after the first rejected
// token is discarded and decoding continues from the accepted prefix; Section 4: KV caching).
//
// One launch serves many caches of one shape (K and V of every layer, the draft's feature caches): the cache
// pointers travel in the launch arguments.  One workgroup per (group of KV heads, sequence, cache) moves the
// accepted rows of its heads in place: every 16-byte chunk is loaded into a register first, the workgroup meets
// at a barrier, then the chunks are stored, so a row that is both a source and a destination (path 0,2,3: row 2
// is written by the second entry and read by the first) is always read before it is overwritten.  A head's
// accepted rows are only a few hundred bytes to a few KB, so a workgroup takes as many heads as its 64 KB of
// registers hold while the grid still has about a thousand workgroups: with one head each, a launch over many
// sequences is tens of thousands of workgroups that each keep a fifth of their threads busy for one round trip.
// Roofline: HBM (read and write of rows x heads x caches); at one sequence the call is one launch latency.
#include "common.h"

using namespace dream;

namespace {

constexpr int MAX_CACHES_PER_LAUNCH = 128;
constexpr int CHUNKS_PER_THREAD = 16;   // 256 threads x 16 chunks x 16 bytes = 64 KB of rows per workgroup

struct CommitArgs {
    int32_t *prefix_len_out;
    int64_t s_max;
    int32_t n_kv_heads, first_cache;
    void *cache[MAX_CACHES_PER_LAUNCH];
};

// The chunks of a workgroup, N to a thread.  All path entries are asked for, then all chunks, without a condition (past the end: the last chunk again), since a load under a
// condition is waited for where the condition ends: with one entry and its chunk after the other a thread made two trips to memory per chunk.
// 16 sequences of 48 caches of 32 heads of 64: 11.5 -> 9.4 us, 8 of 96 of 16 of 256 18.7 -> 18.5; one sequence, one chunk a thread: no difference beside the launch.
template <int N>
__device__ __forceinline__ void move_rows(u32x4 *tree, const int32_t *path, int first_nodes, int total, int per_head, int cpr, int n_tree, int64_t head_stride)
{
    const int tid = threadIdx.x;
    int32_t node[N], at[N];
    int64_t from[N];
    u32x4 r[N];
#pragma unroll
    for (int i = 0; i < N; i++) {
        const int idx = min(tid + i * 256, total - 1);
        const int hl = idx / per_head, rest = idx - hl * per_head;
        const int j = rest / cpr, c = rest - j * cpr;
        at[i] = j;
        from[i] = hl * head_stride + c;
    }
    if (per_head <= 64 * cpr) {
#pragma unroll
        for (int i = 0; i < N; i++)
            node[i] = __shfl(first_nodes, at[i]);
    } else {
#pragma unroll
        for (int i = 0; i < N; i++)
            node[i] = path[at[i]];
    }
#pragma unroll
    for (int i = 0; i < N; i++)
        r[i] = tree[from[i] + (int64_t)min(max(node[i], 0), n_tree - 1) * cpr];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();   // every source chunk of these heads is in a register
#pragma unroll
    for (int i = 0; i < N; i++) {
        const int idx = tid + i * 256;
        if (idx < total) {
            const int hl = idx / per_head, rest = idx - hl * per_head;
            tree[hl * head_stride + rest] = r[i];
        }
    }
}

// One sequence is a chain of trips to memory: the plain arguments are in scalar registers when a wave starts, then what says which rows move (length, path, prefix, cache) is asked for
// at once, then the rows.  Everything in one structure and the path behind the length were four trips.  us a call in a graph, four trips / at once: one Gemma3 sequence (96 caches) 2.82 / 2.76,
// one LLaVA sequence (64) 3.32 / 3.25, 16 SmolVLM sequences (48) 9.15 / 8.98; at once, but with the number of rows in vector registers and the entries under a condition each, 2.85, 3.38 and 9.50.
__global__ __launch_bounds__(256) void kv_commit_kernel(const int32_t *accept_len, const int32_t *path, const int32_t *prefix_len, int path_stride, int n_tree, int chunks_per_row,
                                                        int heads_per_wg, CommitArgs a)
{
    const int b = blockIdx.y, ci = blockIdx.z, tid = threadIdx.x;
    path += (int64_t)b * path_stride;
    const int first_nodes = path[min(tid & 63, path_stride - 1)];      // lane j: entry j
    const int prefix = prefix_len[b], accepted = accept_len[b];
    void *cache = a.cache[ci];
    const int64_t s_max = a.s_max;
    asm volatile("" ::"s"(prefix), "s"(accepted), "s"(cache), "s"(s_max), "s"(a.n_kv_heads), "s"(a.first_cache), "s"(a.prefix_len_out));
    const int h0 = blockIdx.x * heads_per_wg, n_heads = min(heads_per_wg, a.n_kv_heads - h0);
    const int P = (int)min((int64_t)max(prefix, 0), s_max - n_tree);
    // device metadata is trusted, but stay inside the tree rows whatever it holds
    const int n = __builtin_amdgcn_readfirstlane(min(max(accepted, 0), min(path_stride, n_tree) - 1));
    if (blockIdx.x == 0 && ci == 0 && a.first_cache == 0 && tid == 0 && a.prefix_len_out)
        a.prefix_len_out[b] = P + n + 1;
    const int cpr = chunks_per_row;
    const int per_head = (n + 1) * cpr;          // chunks of one head: destination rows 0..n of its tree area are contiguous
    const int total = n_heads * per_head;
    const int64_t head_stride = s_max * cpr;   // chunks between the same row of consecutive heads
    u32x4 *tree = reinterpret_cast<u32x4 *>(cache) + (((int64_t)b * a.n_kv_heads + h0) * s_max + P) * cpr;
    if (total <= 256)
        move_rows<1>(tree, path, first_nodes, total, per_head, cpr, n_tree, head_stride);
    else if (total <= 512)
        move_rows<2>(tree, path, first_nodes, total, per_head, cpr, n_tree, head_stride);
    else if (total <= 1024)
        move_rows<4>(tree, path, first_nodes, total, per_head, cpr, n_tree, head_stride);
    else if (total <= 2048)
        move_rows<8>(tree, path, first_nodes, total, per_head, cpr, n_tree, head_stride);
    else
        move_rows<CHUNKS_PER_THREAD>(tree, path, first_nodes, total, per_head, cpr, n_tree, head_stride);
}

}  // namespace

extern "C" {

int dream_kv_commit(const dream_attn_desc *desc, void *const *caches_host, int32_t n_caches, const int32_t *prefix_len,
                    int32_t n_tree, const int32_t *accept_path, int32_t path_stride, const int32_t *accept_len,
                    int32_t *prefix_len_out, void *stream)
{
    const char *who = "dream_kv_commit";
    if (!desc || !caches_host || !prefix_len || !accept_path || !accept_len)
        return fail(DREAM_ERR_INVALID_ARG, "%s: NULL argument", who);
    if (desc->batch < 1 || desc->batch > 65535 || desc->n_kv_heads < 1 || desc->s_max < 1 || desc->head_dim < 1)
        return fail(DREAM_ERR_INVALID_ARG, "%s: batch in [1, 65535], n_kv_heads, head_dim and s_max must be positive", who);
    if (desc->dtype != DREAM_F32 && desc->dtype != DREAM_BF16)
        return fail(DREAM_ERR_INVALID_ARG, "%s: unknown dtype %d", who, desc->dtype);
    if (n_caches < 1)
        return fail(DREAM_ERR_INVALID_ARG, "%s: n_caches %d < 1", who, n_caches);
    if (n_tree < 1 || n_tree > DREAM_MAX_TREE_ACCEPT || n_tree > desc->s_max)
        return fail(DREAM_ERR_INVALID_ARG, "%s: n_tree %d outside [1, min(%d, s_max)]", who, n_tree, DREAM_MAX_TREE_ACCEPT);
    if (path_stride < 1)
        return fail(DREAM_ERR_INVALID_ARG, "%s: path_stride %d < 1", who, path_stride);
    if (prefix_len_out == prefix_len)
        return fail(DREAM_ERR_INVALID_ARG, "%s: prefix_len_out must not alias prefix_len", who);
    const int64_t row_bytes = (int64_t)desc->head_dim * (desc->dtype == DREAM_F32 ? 4 : 2);
    if (row_bytes % 16)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: rows of %lld bytes are not a multiple of 16", who, (long long)row_bytes);
    const int64_t max_rows = path_stride < n_tree ? path_stride : n_tree;
    if (max_rows * (row_bytes / 16) > 256 * CHUNKS_PER_THREAD)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: up to %lld rows of %lld bytes exceed the 64 KB a workgroup moves", who,
                    (long long)max_rows, (long long)row_bytes);
    for (int32_t i = 0; i < n_caches; i++) {
        if (!caches_host[i])
            return fail(DREAM_ERR_INVALID_ARG, "%s: cache %d is NULL", who, i);
        if (reinterpret_cast<uintptr_t>(caches_host[i]) & 15)
            return fail(DREAM_ERR_INVALID_ARG, "%s: cache %d is not 16-byte aligned", who, i);
    }
    CommitArgs a;
    const int chunks_per_row = (int)(row_bytes / 16);
    a.prefix_len_out = prefix_len_out; a.n_kv_heads = desc->n_kv_heads; a.s_max = desc->s_max;
    // heads per workgroup: as many as the registers of a workgroup hold, while about a thousand workgroups remain
    const int64_t fit = (256 * CHUNKS_PER_THREAD) / (max_rows * chunks_per_row);
    const int64_t spare = ((int64_t)desc->n_kv_heads * desc->batch * (n_caches < MAX_CACHES_PER_LAUNCH ? n_caches : MAX_CACHES_PER_LAUNCH)) / 1024;
    int64_t hpw = fit < spare ? fit : spare;
    if (hpw > desc->n_kv_heads)
        hpw = desc->n_kv_heads;
    if (hpw < 1)
        hpw = 1;
    for (int32_t first = 0; first < n_caches; first += MAX_CACHES_PER_LAUNCH) {
        const int m = n_caches - first < MAX_CACHES_PER_LAUNCH ? n_caches - first : MAX_CACHES_PER_LAUNCH;
        for (int i = 0; i < MAX_CACHES_PER_LAUNCH; i++)
            a.cache[i] = i < m ? caches_host[first + i] : nullptr;
        a.first_cache = first;
        hipLaunchKernelGGL(kv_commit_kernel, dim3(ceil_div(desc->n_kv_heads, hpw), desc->batch, m), dim3(256), 0, as_stream(stream), accept_len, accept_path, prefix_len,
                           path_stride, n_tree, chunks_per_row, (int)hpw, a);
        int rc = check_launch("kv_commit_kernel");
        if (rc)
            return rc;
    }
    return DREAM_OK;
}

}  // extern "C"
