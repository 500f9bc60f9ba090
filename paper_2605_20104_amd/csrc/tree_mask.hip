// graft_build_tree_mask: parent list -> ancestor bitmasks, depths, position ids, leaf paths.
//
// One 128-thread workgroup (two wavefronts) per sequence, one thread per tree
// slot.  The parent list sits in LDS; each thread walks its own ancestor chain
// (at most K steps), so the whole call is a few hundred LDS reads deep and
// launch-latency bound.  Leaves are ranked with a wavefront ballot + popcount and
// write their paths, read off their masks, into a table of bytes in LDS, which goes
// to memory as whole 16-byte groups, each entry stored once.
#include "common.h"

namespace graft {

constexpr int TM_THREADS = GRAFT_MAX_NODES;
constexpr int TM_TABLE = GRAFT_MAX_NODES * GRAFT_MAX_NODES;       // most path entries of a sequence
static_assert(GRAFT_MAX_NODES <= 128, "node indices as signed bytes, two wavefronts");
struct Int4 { int32_t t[4]; };                                    // 16 bytes at any 4-byte boundary

__global__ __launch_bounds__(TM_THREADS) void tree_mask_kernel(
    const int32_t* __restrict__ parent, const int32_t* __restrict__ n_nodes,
    const int32_t* __restrict__ prefix_len, int32_t K_max,
    u64* __restrict__ mask, int32_t* __restrict__ pos, int32_t* __restrict__ depth,
    int32_t* __restrict__ paths, int32_t n_leaf_max, int32_t depth_cap, int32_t* __restrict__ status) {
    const int b = blockIdx.x;
    const int i = threadIdx.x;
    __shared__ int32_t par[TM_THREADS];
    __shared__ int32_t has_child[TM_THREADS];
    __shared__ __attribute__((aligned(16))) signed char table[TM_TABLE];
    __shared__ int32_t or_bad[2], or_over[2];

    const int32_t n = n_nodes[b];
    const int32_t P = prefix_len[b];          // with the other inputs: one trip to memory for all of them
    const bool n_ok = n >= 1 && n <= K_max;
    const int32_t p = i < K_max ? parent[static_cast<size_t>(b) * K_max + i] : -1;
    bool bad = !n_ok;
    if (n_ok && i < n) bad = (i == 0) ? (p != -1) : (p < 0 || p >= i);
    par[i] = p;
    has_child[i] = 0;
    const int32_t width = depth_cap + 1;
    const int32_t entries = paths ? n_leaf_max * width : 0;
    for (int k = 16 * i; k < entries; k += 16 * TM_THREADS)
        *reinterpret_cast<uint4*>(&table[k]) = uint4{~0u, ~0u, ~0u, ~0u};
    const bool any_bad = workgroup_or_128(bad, or_bad);

    int32_t* paths_b = paths ? paths + static_cast<size_t>(b) * entries : nullptr;
    u64* mask_b = mask + static_cast<size_t>(b) * K_max * GRAFT_MASK_WORDS;

    if (any_bad) {
        if (i < K_max) {
            mask_b[i * GRAFT_MASK_WORDS] = 0;
            mask_b[i * GRAFT_MASK_WORDS + 1] = 0;
            pos[static_cast<size_t>(b) * K_max + i] = -1;
            depth[static_cast<size_t>(b) * K_max + i] = -1;
        }
        if (paths_b)
            for (int k = i; k < entries; k += TM_THREADS) paths_b[k] = -1;
        if (i == 0) status[b] = GRAFT_STATUS_BAD_TREE;
        return;
    }

    if (i > 0 && i < n) has_child[p] = 1;              // same value from every writer; read behind the next barrier

    int32_t d = -1;
    unsigned w0 = 0, w1 = 0, w2 = 0, w3 = 0;                  // mask bits 0..31, 32..63, 64..95, 96..127
    if (i < K_max) {
        // (the walk's dependent chain is the LDS read of the parent alone: the mask bits are set in
        //  32-bit words, off that chain)
        if (i < n) {
            for (int32_t j = i; j != -1;) {
                const int32_t up = par[j];
                const unsigned bit = 1u << (j & 31);
                const int word = j >> 5;
                w0 |= word == 0 ? bit : 0u;
                w1 |= word == 1 ? bit : 0u;
                w2 |= word == 2 ? bit : 0u;
                w3 |= word == 3 ? bit : 0u;
                ++d;
                j = up;
            }
        }
        mask_b[i * GRAFT_MASK_WORDS] = (static_cast<u64>(w1) << 32) | w0;
        mask_b[i * GRAFT_MASK_WORDS + 1] = (static_cast<u64>(w3) << 32) | w2;
        depth[static_cast<size_t>(b) * K_max + i] = d;
        pos[static_cast<size_t>(b) * K_max + i] = i < n ? P + d : -1;
    }

    if (!paths_b) {
        if (i == 0) status[b] = 0;
        return;
    }
    // (a node deeper than the cap means a leaf deeper than it)
    const bool too_deep = workgroup_or_128(d > depth_cap, or_over);
    const int lane = i & 63;
    const u64 leaves_lo = __ballot(lane < n && has_child[lane] == 0);             // both wavefronts rank all leaves
    const u64 leaves_hi = __ballot(64 + lane < n && has_child[64 + lane] == 0);
    const u64 own = i < 64 ? leaves_lo : leaves_hi;
    const int32_t rank = __popcll(own & ((1ull << lane) - 1)) + (i < 64 ? 0 : __popcll(leaves_lo));
    if ((own >> lane & 1) != 0 && rank < n_leaf_max && d <= depth_cap) {
        // the path is the mask's bits in increasing order (a parent's index is below its child's)
        signed char* at = table + rank * width;
        const unsigned words[4] = {w0, w1, w2, w3};
#pragma unroll
        for (int w = 0; w < 4; ++w)
            for (unsigned left = words[w]; left != 0; left &= left - 1) *at++ = static_cast<signed char>(32 * w + __builtin_ctz(left));
    }
    __syncthreads();
    for (int k = 4 * i; k + 4 <= entries; k += 4 * TM_THREADS) {
        const int four = *reinterpret_cast<const int*>(&table[k]);
        Int4 out;
#pragma unroll
        for (int u = 0; u < 4; ++u) out.t[u] = static_cast<signed char>(four >> (8 * u));
        *reinterpret_cast<Int4*>(paths_b + k) = out;
    }
    if (i < (entries & 3)) paths_b[(entries & ~3) + i] = table[(entries & ~3) + i];
    if (i == 0)
        status[b] = too_deep || __popcll(leaves_lo) + __popcll(leaves_hi) > n_leaf_max ? GRAFT_STATUS_PATH_OVERFLOW : 0;
}

}  // namespace graft

extern "C" int32_t graft_build_tree_mask(const int32_t* parent, const int32_t* n_nodes,
                                         const int32_t* prefix_len, int32_t B, int32_t K_max,
                                         uint64_t* mask, int32_t* pos, int32_t* depth, int32_t* paths,
                                         int32_t n_leaf_max, int32_t depth_cap, int32_t* status,
                                         void* stream) {
    if (!parent || !n_nodes || !prefix_len || !mask || !pos || !depth || !status) return GRAFT_ERR_NULL;
    if (B < 1 || K_max < 1 || K_max > GRAFT_MAX_NODES) return GRAFT_ERR_SHAPE;
    if (paths && (n_leaf_max < 1 || n_leaf_max > GRAFT_MAX_NODES || depth_cap < 0 ||
                  depth_cap >= GRAFT_MAX_NODES))
        return GRAFT_ERR_SHAPE;
    hipLaunchKernelGGL(graft::tree_mask_kernel, dim3(B), dim3(graft::TM_THREADS), 0,
                       static_cast<hipStream_t>(stream), parent, n_nodes, prefix_len, K_max,
                       reinterpret_cast<graft::u64*>(mask), pos, depth, paths, n_leaf_max, depth_cap,
                       status);
    return graft::check_launch();
}
