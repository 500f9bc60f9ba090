// graft_accept: greedy acceptance walk over the verified hybrid tree.
//
// Two kernels.  In logits mode an argmax kernel scans every node's logits row
// once (an HBM scan: V*4 bytes per node), up to GRAFT_ARGMAX_CHUNKS workgroups per row
// so that even one sequence fills the chip; each writes its chunk's (value,
// first index) to the workspace.  The walk kernel (one 128-thread workgroup per
// sequence, one thread per node) folds the chunk partials into the target's
// greedy token per node, checks each node's whole ancestor chain, and a
// workgroup-wide max over (depth, -index) picks the deepest accepted node.
#include <mutex>

#include "common.h"

namespace graft {

constexpr int AM_THREADS = 256;
constexpr int AM_WAVES = AM_THREADS / 64;
constexpr int AM_QUADS = 12;                     // 16-byte loads in flight per thread: a whole chunk up to V = 196608
static_assert(AM_QUADS * AM_THREADS >= ROW_QUADS, "a chunk of the cut is one round, for V <= 196608");
constexpr int AC_THREADS = GRAFT_MAX_NODES;

struct ArgPartial { float val; int32_t idx; };

// "first maximum": larger value wins, equal values keep the smaller index.
__device__ __forceinline__ void arg_take(float& bv, int32_t& bi, float v, int32_t i) {
    if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
}

// Bound by the logits' way from HBM: a workgroup requests its whole chunk before it looks at any of it, keeps
// only the maximum (one max3 per two elements) and looks for its index in the registers of the lane that
// has it.  8 x 48 rows of 151936 (233 MB): 36 us, 6.5 TB/s; the call, with the walk kernel and the gap before it,
// 48.1 -> 45.4 us, 0.6 of it the walk kernel's; four loads in flight and an (index, value) pair kept per
// element before.
template <bool ONCE>
__global__ __launch_bounds__(AM_THREADS) void argmax_chunk_kernel(
    const float* __restrict__ logits, const int32_t* __restrict__ n_nodes, int32_t K_max, int32_t V,
    int32_t per, ArgPartial* __restrict__ partial) {
    const int chunks = gridDim.x;
    const int chunk = blockIdx.x, i = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x;
    ArgPartial* out = partial + (static_cast<size_t>(b) * K_max + i) * chunks + chunk;
    const int32_t n = n_nodes[b];
    if (i >= n || n > K_max) {                   // padding node: nothing to scan
        if (tid == 0) { out->val = -INFINITY; out->idx = 0x7fffffff; }
        return;
    }
    const float* row = logits + (static_cast<size_t>(b) * K_max + i) * V;
    const RowChunk c = row_chunk(row, V, chunk, chunks, per);
    __shared__ float sv[AM_WAVES + ROW_EDGES];
    __shared__ int32_t si[AM_WAVES + ROW_EDGES];
    if (tid < c.edge) { sv[AM_WAVES + tid] = row[c.edge_at(tid)]; si[AM_WAVES + tid] = c.edge_at(tid); }
    float bv = -INFINITY;                        // the wavefront's maximum so far and its first index
    int32_t bi = 0x7fffffff;
    for (int32_t s0 = c.q0; s0 < c.q1; s0 += AM_QUADS * AM_THREADS) {
        float4 x[AM_QUADS];
#pragma unroll
        for (int u = 0; u < AM_QUADS; ++u) {
            const int32_t qu = s0 + tid + u * AM_THREADS;
            x[u] = qu < c.q1 ? load_logits<ONCE>(c.quad + qu) : float4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        }
        float m = -INFINITY;                     // (fmax passes over NaN, as the comparisons do)
#pragma unroll
        for (int u = 0; u < AM_QUADS; ++u)
            m = __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf(m, x[u].x), __builtin_fmaxf(x[u].y, x[u].z)), x[u].w);
        const float wm = wave_max_f32(m);
        if (wm > bv || bi == 0x7fffffff) {       // uniform over the wavefront
            int32_t at = 0x7fffffff;
            if (m == wm) {                       // hardly ever more than one lane
#pragma unroll
                for (int u = AM_QUADS - 1; u >= 0; --u) {
                    const int32_t qu = s0 + tid + u * AM_THREADS;
                    const int32_t e = c.head + 4 * qu;
                    if (qu < c.q1) {
                        at = x[u].w == wm ? e + 3 : at;
                        at = x[u].z == wm ? e + 2 : at;
                        at = x[u].y == wm ? e + 1 : at;
                        at = x[u].x == wm ? e : at;
                    }
                }
            }
#pragma unroll
            for (int s = 32; s >= 1; s >>= 1) {
                const int32_t other = __shfl_xor(at, s);
                at = other < at ? other : at;
            }
            bv = wm;
            bi = at;
        }
    }
    if ((tid & 63) == 0) { sv[tid >> 6] = bv; si[tid >> 6] = bi; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < AM_WAVES + c.edge; ++w) arg_take(bv, bi, sv[w], si[w]);
        out->val = bv;
        out->idx = bi;
    }
}

// Bound by its chain of dependent steps, so a node's step up the tree is one LDS read: link[j] is j's parent if j
// carries the greedy token of its parent, else -1, and a walk ends at the first mismatch.  Each walk notes the
// nodes it passes as bits; with the best node's bits at hand every node of the path finds its own place (the number of
// bits below it), where one thread used to walk the path again.
__global__ __launch_bounds__(AC_THREADS) void accept_walk_kernel(
    const int32_t* __restrict__ parent, const int32_t* __restrict__ tokens,
    const int32_t* __restrict__ n_nodes, const ArgPartial* __restrict__ partial, int32_t chunks,
    int32_t* __restrict__ target_ids, int32_t K_max, int32_t depth_cap,
    int32_t* __restrict__ accept_len, int32_t* __restrict__ best_node, int32_t* __restrict__ path,
    int32_t* __restrict__ out_tokens, int32_t* __restrict__ status) {
    const int b = blockIdx.x;
    const int i = threadIdx.x;
    __shared__ int32_t tstar[AC_THREADS];
    __shared__ int32_t link[AC_THREADS];
    __shared__ uint4 passed[AC_THREADS];         // nodes on an accepted node's path, as bits
    __shared__ unsigned red[AC_THREADS / 64];
    __shared__ int32_t or_bad[2], or_over[2];

    const int32_t n = n_nodes[b];
    const bool n_ok = n >= 1 && n <= K_max;
    const size_t row = static_cast<size_t>(b) * K_max;
    const int32_t p = i < K_max ? parent[row + i] : -1;
    const int32_t tok = i < K_max ? tokens[row + i] : -1;
    // (requested with the other inputs: one trip to memory for all of them)
    int32_t ts = (!partial && i < K_max) ? target_ids[row + i] : -1;
    // (the scan has written the partials of padding nodes too; requested here and not behind the barrier:
    // 0.6 us less a call)
    ArgPartial pr[GRAFT_ARGMAX_CHUNKS];
    if (partial && i < K_max) {
#pragma unroll
        for (int c = 0; c < GRAFT_ARGMAX_CHUNKS; ++c) pr[c] = partial[(row + i) * chunks + (c < chunks ? c : 0)];   // (one read again does no harm)
    }
    bool bad = !n_ok;
    if (n_ok && i < n) bad = (i == 0) ? (p != -1) : (p < 0 || p >= i);
    // the target's greedy token after each node
    if (partial && i < K_max && i < n) {
        float bv = pr[0].val;
        int32_t bi = pr[0].idx;
#pragma unroll
        for (int c = 1; c < GRAFT_ARGMAX_CHUNKS; ++c) arg_take(bv, bi, pr[c].val, pr[c].idx);
        ts = bi;
    }
    tstar[i] = ts;
    const bool any_bad = workgroup_or_128(bad, or_bad);

    const int32_t width = depth_cap + 1;
    int32_t* path_b = path + static_cast<size_t>(b) * width;
    int32_t* out_b = out_tokens + static_cast<size_t>(b) * width;
    if (any_bad) {
        for (int k = i; k < width; k += AC_THREADS) { path_b[k] = -1; out_b[k] = -1; }
        if (partial && i < K_max) target_ids[row + i] = -1;
        if (i == 0) { accept_len[b] = 0; best_node[b] = -1; status[b] = GRAFT_STATUS_BAD_TREE; }
        return;
    }
    if (partial && i < K_max) target_ids[row + i] = ts;
    link[i] = (i > 0 && i < n && tok == tstar[p]) ? p : -1;
    __syncthreads();

    // accepted iff every node on the path below the root carries its parent's greedy token
    bool ok = i < n;
    int32_t d = 0;
    uint4 bits = uint4{1u, 0u, 0u, 0u};          // the root
    if (ok) {
        int32_t j = i;
        while (j > 0) {
            const int32_t up = link[j];
            const unsigned bit = 1u << (j & 31);
            const int word = j >> 5;
            bits.x |= word == 0 ? bit : 0u;
            bits.y |= word == 1 ? bit : 0u;
            bits.z |= word == 2 ? bit : 0u;
            bits.w |= word == 3 ? bit : 0u;
            ++d;
            j = up;
        }
        ok = j == 0;
    }
    passed[i] = bits;
    const int over = (ok && d > depth_cap) ? 1 : 0;
    // key: depth first, then smaller index; 0 = not a candidate (the root gives key >= 1)
    const unsigned key = (ok && d <= depth_cap) ? ((static_cast<unsigned>(d) << 8) | static_cast<unsigned>(255 - i)) : 0u;
    const unsigned wmax = wave_max_u32(key);
    if ((i & 63) == 0) red[i >> 6] = wmax;
    const bool any_over = workgroup_or_128(over != 0, or_over);
    const unsigned best = red[0] > red[1] ? red[0] : red[1];
    const int32_t best_i = 255 - static_cast<int32_t>(best & 255u), best_d = static_cast<int32_t>(best >> 8);
    const uint4 on = passed[best_i];
    const unsigned words[4] = {on.x, on.y, on.z, on.w};
    int32_t k = 0;                               // nodes of the path before this one
    bool mine = false;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int32_t at = i - 32 * w;
        k += __popc(at >= 32 ? words[w] : (at > 0 ? words[w] & ((1u << at) - 1u) : 0u));
        if (at >= 0 && at < 32) mine = (words[w] >> at) & 1u;
    }
    if (mine) {                                  // (best_d <= depth_cap)
        path_b[k] = i;
        if (k > 0) out_b[k - 1] = tok;
    }
    if (i == best_i) {
        accept_len[b] = best_d;
        best_node[b] = i;
        status[b] = any_over ? GRAFT_STATUS_PATH_OVERFLOW : 0;
        out_b[best_d] = ts;
    }
    // the padding behind the path: all threads, not one after the other
    for (int32_t q = best_d + 1 + i; q < width; q += AC_THREADS) { path_b[q] = -1; out_b[q] = -1; }
}

// ---- graft_accept_noalloc: the argmax partials live in a file-scope device array ----------
// In host code the array's name is only a stand-in for the symbol: the device address is
// asked for once per device (hipGetSymbolAddress with that device current; every GPU holds its
// own copy at its own address) and that pointer is what the kernels get.
constexpr int NA_MAX_ROWS = GRAFT_NOALLOC_MAX_ROWS;   // B * K_max logits rows per call
constexpr int NA_MAX_DEVICES = 64;
static __device__ __align__(256) unsigned char scratch[static_cast<size_t>(NA_MAX_ROWS) * GRAFT_ARGMAX_CHUNKS *
                                                       sizeof(ArgPartial)];   // 1 MiB
static void* g_scratch_ptr[NA_MAX_DEVICES];
static std::mutex g_scratch_lock;

// Device address of `scratch` on the current device, or nullptr (with the HIP error recorded).
static ArgPartial* scratch_on_current_device() {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess && (dev < 0 || dev >= NA_MAX_DEVICES)) e = hipErrorInvalidDevice;
    if (e == hipSuccess) {
        std::lock_guard<std::mutex> hold(g_scratch_lock);
        if (!g_scratch_ptr[dev]) {
            void* ptr = nullptr;
            e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (e == hipSuccess && !ptr) e = hipErrorInvalidSymbol;
            if (e == hipSuccess) g_scratch_ptr[dev] = ptr;
        }
        if (e == hipSuccess) return static_cast<ArgPartial*>(g_scratch_ptr[dev]);
    }
    (void)hipGetLastError();
    set_last_hip_error(static_cast<int32_t>(e));
    return nullptr;
}

static int32_t accept_impl(const int32_t* parent, const int32_t* tokens, const int32_t* n_nodes,
                           const float* logits, int32_t V, int32_t* target_ids, int32_t B, int32_t K_max,
                           int32_t depth_cap, int32_t* accept_len, int32_t* best_node, int32_t* path,
                           int32_t* out_tokens, int32_t* status, ArgPartial* ws, hipStream_t s) {
    const ArgPartial* partial = nullptr;
    int32_t chunks = 0;
    if (logits) {
        const RowCut cut = row_cut(static_cast<int64_t>(B) * K_max, V);
        chunks = cut.chunks;
        const auto scan = read_once(static_cast<int64_t>(B) * K_max, V) ? argmax_chunk_kernel<true> : argmax_chunk_kernel<false>;
        hipLaunchKernelGGL(scan, dim3(chunks, K_max, B), dim3(AM_THREADS), 0, s, logits, n_nodes, K_max, V, cut.per, ws);
        int32_t rc = check_launch();
        if (rc != GRAFT_OK) return rc;
        partial = ws;
    }
    hipLaunchKernelGGL(accept_walk_kernel, dim3(B), dim3(AC_THREADS), 0, s, parent, tokens, n_nodes, partial,
                       chunks, target_ids, K_max, depth_cap, accept_len, best_node, path, out_tokens, status);
    return check_launch();
}

static int32_t accept_args_ok(const int32_t* parent, const int32_t* tokens, const int32_t* n_nodes,
                              const int32_t* target_ids, int32_t B, int32_t K_max, int32_t depth_cap,
                              const int32_t* accept_len, const int32_t* best_node, const int32_t* path,
                              const int32_t* out_tokens, const int32_t* status) {
    if (!parent || !tokens || !n_nodes || !target_ids || !accept_len || !best_node || !path ||
        !out_tokens || !status)
        return GRAFT_ERR_NULL;
    if (B < 1 || B > 65535 || K_max < 1 || K_max > GRAFT_MAX_NODES || depth_cap < 0 ||
        depth_cap >= GRAFT_MAX_NODES)
        return GRAFT_ERR_SHAPE;
    return GRAFT_OK;
}

}  // namespace graft

extern "C" size_t graft_accept_workspace_bytes(int32_t B, int32_t K_max, int32_t V) {
    if (B < 1 || K_max < 1 || V < 1) return 0;
    return static_cast<size_t>(B) * K_max * GRAFT_ARGMAX_CHUNKS * sizeof(graft::ArgPartial);
}

extern "C" int32_t graft_accept(const int32_t* parent, const int32_t* tokens, const int32_t* n_nodes,
                                const float* logits, int32_t V, int32_t* target_ids, int32_t B,
                                int32_t K_max, int32_t depth_cap, int32_t* accept_len,
                                int32_t* best_node, int32_t* path, int32_t* out_tokens, int32_t* status,
                                void* workspace, size_t workspace_bytes, void* stream) {
    const int32_t rc = graft::accept_args_ok(parent, tokens, n_nodes, target_ids, B, K_max, depth_cap, accept_len,
                                             best_node, path, out_tokens, status);
    if (rc != GRAFT_OK) return rc;
    if (logits) {
        if (V < 1) return GRAFT_ERR_SHAPE;
        if (!workspace || workspace_bytes < graft_accept_workspace_bytes(B, K_max, V))
            return GRAFT_ERR_WORKSPACE;
    }
    return graft::accept_impl(parent, tokens, n_nodes, logits, V, target_ids, B, K_max, depth_cap, accept_len,
                              best_node, path, out_tokens, status, static_cast<graft::ArgPartial*>(workspace),
                              static_cast<hipStream_t>(stream));
}

extern "C" int32_t graft_accept_noalloc(const int32_t* parent, const int32_t* tokens, const int32_t* n_nodes,
                                        const float* logits, int32_t V, int32_t* target_ids, int32_t B,
                                        int32_t K_max, int32_t depth_cap, int32_t* accept_len,
                                        int32_t* best_node, int32_t* path, int32_t* out_tokens,
                                        int32_t* status, void* stream) {
    const int32_t rc = graft::accept_args_ok(parent, tokens, n_nodes, target_ids, B, K_max, depth_cap, accept_len,
                                             best_node, path, out_tokens, status);
    if (rc != GRAFT_OK) return rc;
    graft::ArgPartial* ws = nullptr;
    if (logits) {
        if (V < 1) return GRAFT_ERR_SHAPE;
        if (static_cast<int64_t>(B) * K_max > graft::NA_MAX_ROWS) return GRAFT_ERR_WORKSPACE;   // beyond the static scratch
        ws = graft::scratch_on_current_device();
        if (!ws) return GRAFT_ERR_HIP;
    }
    return graft::accept_impl(parent, tokens, n_nodes, logits, V, target_ids, B, K_max, depth_cap, accept_len,
                              best_node, path, out_tokens, status, ws, static_cast<hipStream_t>(stream));
}
