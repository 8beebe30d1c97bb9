// dream_accept_path: per-node arg-max over the vocabulary and the greedy accepted path.
//
// At temperature 0 the acceptance rule of Section 2.1 accepts a drafted token exactly when it is
// the target's arg-max at its parent; everything after the first mismatch on a path is dropped and
// the target's own choice at the last accepted node is emitted as the bonus token (Section 4).
//
// argmax_partial_kernel streams the logits once (16-byte loads, one workgroup per row chunk) and
// reduces (value, index) pairs to one 64-bit key per chunk; ties always keep the lower
// index, so the result does not depend on how rows are chunked.  accept_walk_kernel, one workgroup per sequence, merges
// the chunk keys of a node with adjacent lanes; then one wave lets every node check its own path to the root.
#include "common.h"
#include <type_traits>
#include <mutex>

using namespace dream;

// Scratch of dream_accept_path_static: the per-chunk keys live here instead of in a
// caller's workspace.  One copy per GPU, held until the process ends; host code only ever uses the address
// hipGetSymbolAddress reports for the current device, never the symbol itself.
static __device__ __align__(256) unsigned char scratch[DREAM_ACCEPT_STATIC_SCRATCH_BYTES];

namespace {

constexpr int CHUNK_ELEMS = 8192;   // logits handled by one workgroup
constexpr int MAX_DEVICES = 64;

// (value, index) as one integer whose order is "larger value, then lower index"
__device__ __forceinline__ uint64_t make_key(float v, int i)
{
    v += 0.0f;   // -0 and +0 are equal values
    const uint32_t u = __float_as_uint(v);
    return ((uint64_t)((u & 0x80000000u) ? ~u : (u | 0x80000000u)) << 32) | (0xffffffffu - (uint32_t)i);
}

// The smallest index of the wave, in every lane.
__device__ __forceinline__ int wave_min(int v)
{
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false));   // row_ror:8, 4, 2, 1
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x124, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x122, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x121, 0xf, 0xf, false));
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)), min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// Bound by the reading of the logits where there are many, by latency otherwise.  A thread asks for all of its 16-byte pieces at once, takes the maximum of each and looks for the
// index only in the first piece that holds the wave's maximum: before, it waited for one piece after the other and compared element by
// element.  Calls, us, before / now (both kernels): 60 rows of 262144 bf16 logits 13.1 / 11.0, of 32000 9.7 / 6.1, 16 x 60 of 49152 22.5 / 19.6, 4 x 33 of 131072 float32 21.0 / 15.8;
// rows of odd lengths, which came one logit at a time: 60 of 32003 bf16 11.7 to 12.9 / 7.9, 8 x 60 of 50257 float32 43.6 / 21.0.
template <bool BF16>
__global__ __launch_bounds__(256) void argmax_partial_kernel(const void *logits, int vocab, int n_chunks, uint64_t *part)
{
    constexpr int PER = BF16 ? 8 : 4, PIECES = CHUNK_ELEMS / (256 * PER);     // logits of a piece, pieces of a thread
    const int chunk = blockIdx.x;
    const int64_t row = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int begin = chunk * CHUNK_ELEMS;
    const int end = min(begin + CHUNK_ELEMS, vocab);
    const char *p = reinterpret_cast<const char *>(logits) + (row * vocab + begin) * (BF16 ? 2 : 4);
    // whole pieces in 16-byte loads, which global memory serves from any address of a logit, the tail one by one
    const int n_vec = (end - begin) / PER;
    float best = -INFINITY, m;
    int best_i = 0x7fffffff, index;
    auto at = [&](int j) { return min(j * 256 + tid, n_vec - 1); };           // past the last piece: that one again
    auto element = [&](const u32x4 &v, int e) { return __uint_as_float(!BF16 ? v[e] : e & 1 ? v[e / 2] & 0xffff0000u : v[e / 2] << 16); };
    // the wave's maximum and the first index that has it, from N pieces of every thread and the tail
    auto search = [&](auto pieces) {
        constexpr int N = decltype(pieces)::value;
        u32x4 w[N];
        float piece_max[N];
        m = -INFINITY;
        if (n_vec > 0) {
#pragma unroll
            for (int j = 0; j < N; j++) {
                const u32x4_any *from = reinterpret_cast<const u32x4_any *>(p) + at(j);
                w[j] = BF16 ? __builtin_nontemporal_load(from) : *from;       // bf16 logits: read once
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < N; j++) {
                float x = -INFINITY;
#pragma unroll
                for (int e = 0; e < PER; e++)
                    x = fmaxf(x, __builtin_canonicalizef(element(w[j], e)));  // passes a NaN over (a signalling one would take the maximum so far with it)
                piece_max[j] = x;
                m = fmaxf(m, x);
            }
        }
        for (int i = begin + n_vec * PER + tid; i < end; i += 256) {
            const float x = BF16 ? bf16_bits_to_float(reinterpret_cast<const uint16_t *>(p)[i - begin]) : reinterpret_cast<const float *>(p)[i - begin];
            if (x > best || (x == best && i < best_i)) { best = x; best_i = i; }
        }
        m = fmaxf(m, best);
        m = wave_max(m);
        index = m > -INFINITY ? (best == m ? best_i : 0x7fffffff) : begin;    // nothing above -inf: the chunk's first, so that a fully masked row has index 0
        if (n_vec > 0 && m > -INFINITY) {
            // the thread's first piece with the maximum, the first logit of it (the pieces lie before the tail)
            u32x4 first = {0, 0, 0, 0};
            int from = -1;
#pragma unroll
            for (int j = N - 1; j >= 0; j--)
                if (piece_max[j] == m) {
                    first = w[j];
                    from = at(j);
                }
            if (from >= 0) {
#pragma unroll
                for (int e = PER - 1; e >= 0; e--)
                    index = element(first, e) == m ? begin + from * PER + e : index;
            }
        }
    };
    // Only as many pieces as the chunk has: with all of them for a short row its pieces were asked for again and again.  Calls, us, all / as many: 17 x 239 rows of 1000 bf16 logits 12.8 / 10.5,
    // 26 x 135 of 300 float32 11.6 / 8.9, 40 x 48 of 2000 bf16 8.5 / 7.6, 60 x 60 of 3000 float32 11.5 / 11.0.
    if (n_vec <= 256)
        search(std::integral_constant<int, 1>{});
    else if (n_vec <= 256 * PIECES / 2)
        search(std::integral_constant<int, PIECES / 2>{});
    else
        search(std::integral_constant<int, PIECES>{});
    index = wave_min(index);
    __shared__ uint64_t s_key[4];
    if (lane == 0)
        s_key[wave] = make_key(m, index);
    __syncthreads();
    if (tid == 0) {
        uint64_t key = s_key[0];
        for (int w = 1; w < 4; w++)
            key = s_key[w] > key ? s_key[w] : key;
        part[row * n_chunks + chunk] = key;
    }
}

// The largest key of `lanes` adjacent lanes (a power of two, the same in the whole wave) in all of them, by register moves.  (Shuffles are trips through LDS, one after the other: calls in a
// graph, 60 nodes of 32 chunks 9.2 us, 8.4 so; 16 sequences of 60 nodes of 6 chunks 17.9, 17.4 so.)
template <int CTRL>
__device__ __forceinline__ uint64_t max_with(uint64_t k)
{
    const uint32_t lo = __builtin_amdgcn_update_dpp(0u, (uint32_t)k, CTRL, 0xf, 0xf, false), hi = __builtin_amdgcn_update_dpp(0u, (uint32_t)(k >> 32), CTRL, 0xf, 0xf, false);
    const uint64_t o = (uint64_t)hi << 32 | lo;
    return o > k ? o : k;
}
__device__ __forceinline__ uint64_t max_of_lanes(uint64_t k, int lanes)
{
    if (lanes > 1)
        k = max_with<0xb1>(k);       // quad_perm 1, 0, 3, 2
    if (lanes > 2)
        k = max_with<0x4e>(k);       // quad_perm 2, 3, 0, 1
    if (lanes > 4)
        k = max_with<0x141>(k);      // row_half_mirror: the other four of eight lanes, which hold one value each
    if (lanes > 8)
        k = max_with<0x140>(k);      // row_mirror: the other eight
    if (lanes > 16) {                // the rows of 16 lanes, even ones in one result and odd ones in the other
        const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)k, (uint32_t)k, false, false), hi = __builtin_amdgcn_permlane16_swap((uint32_t)(k >> 32), (uint32_t)(k >> 32), false, false);
        const uint64_t a = (uint64_t)hi[0] << 32 | lo[0], b = (uint64_t)hi[1] << 32 | lo[1];
        k = a > b ? a : b;
    }
    if (lanes > 32) {
        const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)k, (uint32_t)k, false, false), hi = __builtin_amdgcn_permlane32_swap((uint32_t)(k >> 32), (uint32_t)(k >> 32), false, false);
        const uint64_t a = (uint64_t)hi[0] << 32 | lo[0], b = (uint64_t)hi[1] << 32 | lo[1];
        k = a > b ? a : b;
    }
    return k;
}

// One workgroup per sequence.  `lanes` adjacent lanes (a power of two) merge the chunk results of a node; then one wave lets every
// node check its own root path (a node is accepted iff every edge above it matches the target's arg-max and it is not deeper
// than max_depth); the deepest accepted node, lowest index among equals, wins a wave reduction; lane 0 writes its path.  Trees of up to 64 nodes go down
// level by level instead, a lane per node and a ballot per level, and up the path by lane reads: no chains of LDS reads.
// Latency bound.  Measured, 60 nodes of 32 chunks: 7.8 us with one wave that read a node's chunks one lane each, 5.6 us with 512 threads, less by 1 to 2 us with these and with the
// parents and tokens asked for beside the keys (the call with 60 nodes of 4 chunks: 9.7 / 6.1 us, with 200 nodes 11.1 / 9.8).
constexpr int WALK = 512;

__global__ __launch_bounds__(WALK) void accept_walk_kernel(const uint64_t *part, int n_chunks, int lanes, int n_tree, const int32_t *token,
                                                           const int32_t *parent, int max_depth, int32_t *node_argmax, int32_t *accept_len,
                                                           int32_t *accept_path, int32_t *bonus_token)
{
    __shared__ int32_t s_am[DREAM_MAX_TREE_ACCEPT];
    __shared__ int32_t s_par[DREAM_MAX_TREE_ACCEPT];
    __shared__ int32_t s_tok[DREAM_MAX_TREE_ACCEPT];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int64_t bt = (int64_t)b * n_tree;
    const int sub = tid & (lanes - 1), per_pass = WALK / lanes;
    constexpr int U = 4;                 // passes whose loads are in flight together
    const int own = min(tid, n_tree - 1);
    int par_own = -1, tok_own = 0;       // of node tid
    for (int i0 = tid / lanes; __any(i0 < n_tree); i0 += U * per_pass) {
        uint64_t best[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int i = min(i0 + u * per_pass, n_tree - 1);
            best[u] = part[(bt + i) * n_chunks + min(sub, n_chunks - 1)];
        }
        par_own = parent[bt + own];      // here, so that no wait for them stands before the keys are asked for
        tok_own = token[bt + own];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int i = i0 + u * per_pass;
            for (int ch = sub + lanes; i < n_tree && ch < n_chunks; ch += lanes) {
                const uint64_t o = part[(bt + i) * n_chunks + ch];
                best[u] = o > best[u] ? o : best[u];
            }
        }
        if (lanes > 1)
#pragma unroll
            for (int u = 0; u < U; u++)
                best[u] = max_of_lanes(best[u], lanes);
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int i = i0 + u * per_pass;
            if (i < n_tree && sub == 0) {
                const int idx = (int)(0xffffffffu - (uint32_t)best[u]);
                s_am[i] = idx;
                node_argmax[bt + i] = idx;
            }
        }
    }
    if (tid < n_tree) {                  // (its wave has been in the loop: lanes that share a node make no more than one node of a thread)
        s_par[tid] = par_own < tid ? par_own : -1;   // a walk up the tree always ends
        s_tok[tid] = tok_own;
    }
    for (int i = tid + WALK; i < n_tree; i += WALK) {
        const int par = parent[bt + i];
        s_par[i] = par < i ? par : -1;
        s_tok[i] = token[bt + i];
    }
    __syncthreads();
    if (tid >= 64)
        return;
    int32_t *path = accept_path + (int64_t)b * (max_depth + 1);
    if (n_tree <= 64) {
        // lane i is node i: the accepted nodes of a level are those whose parent is one of the level before
        const int par = lane > 0 && lane < n_tree && par_own < lane ? par_own : -1;
        const bool fits = par >= 0 && tok_own == s_am[max(par, 0)];
        uint64_t level = 1ull;
        int depth = 0;
        while (depth < max_depth) {
            const uint64_t next = __ballot(fits && (level >> par & 1));
            if (!next)
                break;
            level = next;
            depth++;
        }
        const int deepest = __builtin_ctzll(level);
        for (int t = depth + 1 + lane; t <= max_depth; t += 64)
            path[t] = -1;
        int n = deepest, mine = 0;       // lane t: node t of the path
        for (int t = depth; t > 0; t--) {
            mine = lane == t ? n : mine;
            n = __builtin_amdgcn_readlane(par, n);
        }
        if (lane <= depth)
            path[lane] = mine;
        if (lane == 0) {
            accept_len[b] = depth;
            bonus_token[b] = s_am[deepest];
        }
        return;
    }
    int best_d = -1, best_i = 0x7fffffff;
    for (int i = lane; i < n_tree; i += 64) {
        int d = 0;
        bool ok = true;
        for (int a = i; a > 0 && ok; d++) {
            const int p = s_par[a];
            ok = p >= 0 && s_tok[a] == s_am[p];
            a = p;
        }
        if (ok && d <= max_depth && d > best_d) {   // nodes are visited in increasing index: strict '>' keeps the lowest
            best_d = d;
            best_i = i;
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const int od = __shfl_xor(best_d, off), oi = __shfl_xor(best_i, off);
        if (od > best_d || (od == best_d && oi < best_i)) {
            best_d = od;
            best_i = oi;
        }
    }
    if (lane == 0) {
        accept_len[b] = best_d;
        for (int t = best_d + 1; t <= max_depth; t++)
            path[t] = -1;
        int d = best_d;
        for (int n = best_i; n >= 0 && d >= 0; n = s_par[n])
            path[d--] = n;
        bonus_token[b] = s_am[best_i];
    }
}

size_t partial_bytes(int batch, int n_tree, int vocab)
{
    const size_t n = (size_t)batch * n_tree * ceil_div(vocab, CHUNK_ELEMS);
    return align_up(n * 4, 256) + align_up(n * 4, 256);
}

int validate_accept(const char *who, const void *logits, int logits_dtype, int batch, int n_tree, int vocab, const int32_t *token,
                    const int32_t *parent, int max_depth, const int32_t *node_argmax, const int32_t *accept_len,
                    const int32_t *accept_path, const int32_t *bonus_token)
{
    if (!logits || !token || !parent || !node_argmax || !accept_len || !accept_path || !bonus_token)
        return fail(DREAM_ERR_INVALID_ARG, "%s: NULL argument", who);
    if (logits_dtype != DREAM_F32 && logits_dtype != DREAM_BF16)
        return fail(DREAM_ERR_INVALID_ARG, "%s: unknown logits dtype %d", who, logits_dtype);
    if (batch < 1 || vocab < 1 || max_depth < 0)
        return fail(DREAM_ERR_INVALID_ARG, "%s: batch, vocab must be positive and max_depth non-negative", who);
    if (n_tree < 1 || n_tree > DREAM_MAX_TREE_ACCEPT)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: n_tree %d outside [1, %d]", who, n_tree, DREAM_MAX_TREE_ACCEPT);
    if ((int64_t)batch * n_tree > 65535)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: batch * n_tree = %lld exceeds 65535 rows", who, (long long)batch * n_tree);
    return DREAM_OK;
}

// The two launches; `partials` is device memory of partial_bytes() bytes (a workspace or the static scratch).
int launch_accept(const void *logits, int logits_dtype, int batch, int n_tree, int vocab, const int32_t *token, const int32_t *parent,
                  int max_depth, int32_t *node_argmax, int32_t *accept_len, int32_t *accept_path, int32_t *bonus_token, void *partials,
                  void *stream)
{
    const int n_chunks = ceil_div(vocab, CHUNK_ELEMS);
    uint64_t *part = static_cast<uint64_t *>(partials);
    int lanes = 1;
    while (lanes < n_chunks && lanes < 64)
        lanes *= 2;
    hipStream_t st = as_stream(stream);
    dim3 grid(n_chunks, batch * n_tree);
    if (logits_dtype == DREAM_BF16)
        hipLaunchKernelGGL(argmax_partial_kernel<true>, grid, dim3(256), 0, st, logits, vocab, n_chunks, part);
    else
        hipLaunchKernelGGL(argmax_partial_kernel<false>, grid, dim3(256), 0, st, logits, vocab, n_chunks, part);
    int rc = check_launch("argmax_partial_kernel");
    if (rc)
        return rc;
    hipLaunchKernelGGL(accept_walk_kernel, dim3(batch), dim3(WALK), 0, st, part, n_chunks, lanes, n_tree, token, parent, max_depth, node_argmax,
                       accept_len, accept_path, bonus_token);
    return check_launch("accept_walk_kernel");
}

// Device address of `scratch` on the current GPU, looked up once per device (each GPU holds its own copy).
int static_scratch_address(const char *who, void **out)
{
    static std::mutex mu;
    static void *address[MAX_DEVICES] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES)
        return fail(DREAM_ERR_HIP, "%s: no current HIP device (or its index is not below %d)", who, MAX_DEVICES);
    std::lock_guard<std::mutex> lock(mu);
    if (!address[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(DREAM_ERR_HIP, "%s: hipGetSymbolAddress(scratch) on device %d: %s", who, dev, hipGetErrorString(e));
        address[dev] = p;
    }
    *out = address[dev];
    return DREAM_OK;
}

}  // namespace

extern "C" {

size_t dream_accept_path_workspace(int32_t batch, int32_t n_tree, int32_t vocab)
{
    if (batch < 1 || n_tree < 1 || vocab < 1)
        return DREAM_WORKSPACE_MIN_BYTES;
    return DREAM_WORKSPACE_MIN_BYTES + partial_bytes(batch, n_tree, vocab);
}

int dream_accept_path(const void *logits, int32_t logits_dtype, int32_t batch, int32_t n_tree, int32_t vocab,
                      const int32_t *token, const int32_t *parent, int32_t max_depth, int32_t *node_argmax,
                      int32_t *accept_len, int32_t *accept_path, int32_t *bonus_token, void *workspace,
                      size_t workspace_bytes, void *stream)
{
    const char *who = "dream_accept_path";
    int rc = validate_accept(who, logits, logits_dtype, batch, n_tree, vocab, token, parent, max_depth, node_argmax, accept_len,
                             accept_path, bonus_token);
    if (rc)
        return rc;
    const size_t need = dream_accept_path_workspace(batch, n_tree, vocab);
    if (!workspace || workspace_bytes < need)
        return fail(DREAM_ERR_WORKSPACE, "%s: workspace of %zu bytes, %zu needed", who, workspace_bytes, need);
    return launch_accept(logits, logits_dtype, batch, n_tree, vocab, token, parent, max_depth, node_argmax, accept_len, accept_path,
                         bonus_token, static_cast<char *>(workspace) + DREAM_WORKSPACE_MIN_BYTES, stream);
}

int dream_accept_path_static(const void *logits, int32_t logits_dtype, int32_t batch, int32_t n_tree, int32_t vocab,
                             const int32_t *token, const int32_t *parent, int32_t max_depth, int32_t *node_argmax,
                             int32_t *accept_len, int32_t *accept_path, int32_t *bonus_token, void *stream)
{
    const char *who = "dream_accept_path_static";
    int rc = validate_accept(who, logits, logits_dtype, batch, n_tree, vocab, token, parent, max_depth, node_argmax, accept_len,
                             accept_path, bonus_token);
    if (rc)
        return rc;
    const size_t need = partial_bytes(batch, n_tree, vocab);
    if (need > DREAM_ACCEPT_STATIC_SCRATCH_BYTES)
        return fail(DREAM_ERR_UNSUPPORTED, "%s: batch * n_tree * ceil(vocab / %d) = %zu partial results need %zu bytes, the static scratch "
                    "holds %d; use dream_accept_path with a workspace", who, CHUNK_ELEMS,
                    (size_t)batch * n_tree * ceil_div(vocab, CHUNK_ELEMS), need, DREAM_ACCEPT_STATIC_SCRATCH_BYTES);
    void *base = nullptr;
    rc = static_scratch_address(who, &base);
    if (rc)
        return rc;
    // every partial result the walk reads is written by this call's first kernel: nothing has to start at zero
    return launch_accept(logits, logits_dtype, batch, n_tree, vocab, token, parent, max_depth, node_argmax, accept_len, accept_path,
                         bonus_token, base, stream);
}

int dream_accept_static_init(void)
{
    void *base = nullptr;
    return static_scratch_address("dream_accept_static_init", &base);
}

}  // extern "C"
