// graft_kv_compact: after acceptance the accepted path's keys and values move from their
// tree slots to the positions right behind the prefix, in every layer's paged cache.
//
// The rows to move are few (accept_len * Hkv * D elements per layer and side), so the call is
// a scatter of short copies, bound by its chain of dependent trips to memory: lengths and path, page table,
// rows.  Every wavefront works for itself, without LDS or a barrier: lane l stands for the rows l + 1 and l + 65 of
// the path, which it requests together with the lengths, checks, and looks up in the page table; the copy loop takes
// the addresses from the lanes.  (One thread of a workgroup used to check the path entry by entry, between two
// barriers, and the path was requested behind the lengths: 32 layers of 8 heads of 128 in bf16, 4 rows, one sequence 4.75 us a
// call in a graph, 3.82 like this; 2.95 with the rows of a batch in registers, see Quad.)
// One lane of the copy owns one 16-byte column of a token row (a fixed KV head and element range)
// for one sequence and layer and walks the path in order, eight rows at a time: all eight
// (K and V: sixteen loads) are in flight before the first store.  Doing this in place is safe because the path
// increases strictly: position P + k is written by the thread that alone uses this column, and only after it
// has read every source P + path[k'] with k' <= k + 7; later sources lie beyond P + k + 7.
#include "common.h"

namespace graft {

// Wavefronts share nothing, and a workgroup is one as long as all of them start at once.  Past that their number costs: 4096
// wavefronts of 64 layers and 16 sequences that move nothing take 3.5 us one by one, 2.4 four to a workgroup.  (One long
// path in 48 layers of 8 heads in fp32, 192 wavefronts, the other way round: 9.4 us one by one, 11.3 four to a workgroup.)
constexpr int KC_THREADS = 256;
constexpr int64_t KC_ALONE = 1024;               // wavefronts of a launch up to which each is a workgroup
constexpr int KC_BATCH = 8;
static_assert(64 % KC_BATCH == 0 && GRAFT_MAX_NODES <= 128, "a batch stays within one register of the lanes' rows");

// 16 bytes as the compiler's own vector: arrays of HIP's uint4, a class, went to scratch memory (272 bytes a lane), there and back
// for each row.  us a call in a graph, one sequence, 32 layers of 8 heads of 128 in bf16, 4 / 48 rows 3.82 / 15.4 -> 2.95 / 7.8; 16
// sequences, 48 layers in fp32, 20.6 / 181 -> 8.7 / 99.
typedef unsigned Quad __attribute__((ext_vector_type(4)));

struct CompactParams {
    void* k;
    void* v;
    int32_t* new_prefix_len;
    int32_t* status;
    int64_t layer_stride, page_stride, token_stride, head_stride;   // in elements
    int32_t Hkv, elem_shift, cols_shift;
};

// (the arguments of the first two trips stand first: they arrive in registers)
__global__ __launch_bounds__(KC_THREADS) void kv_compact_kernel(
    const int32_t* __restrict__ prefix_len, const int32_t* __restrict__ accept_len, const int32_t* __restrict__ path,
    const int32_t* __restrict__ block_table, int32_t depth_cap, int32_t K_max, int32_t max_pages, CompactParams p) {
    const int b = blockIdx.z, layer = blockIdx.y, lane = threadIdx.x & 63;
    const int32_t* path_b = path + static_cast<size_t>(b) * (depth_cap + 1);
    const int32_t P = __builtin_amdgcn_readfirstlane(prefix_len[b]), a = __builtin_amdgcn_readfirstlane(accept_len[b]);
    const int32_t first = path_b[0];
    int32_t node[2], above[2];                   // path[k] and path[k - 1] of this lane's rows k
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int32_t k = lane + 1 + 64 * h;
        node[h] = path_b[k < depth_cap ? k : depth_cap];
        above[h] = path_b[k - 1 < depth_cap ? k - 1 : depth_cap];
    }
    bool bad = first != 0, outside = false;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const bool used = lane + 1 + 64 * h <= a;
        bad = bad || (used && (node[h] <= above[h] || node[h] >= K_max));
        outside = outside || (used && static_cast<int64_t>(P) + node[h] >= static_cast<int64_t>(max_pages) * GRAFT_PAGE_SIZE);
    }
    int32_t st = 0;
    if (P < 0 || a < 0 || a > depth_cap) st = GRAFT_STATUS_BAD_LENGTH;
    else if (__builtin_amdgcn_ballot_w64(bad) != 0) st = GRAFT_STATUS_BAD_TREE;
    else if (__builtin_amdgcn_ballot_w64(outside) != 0) st = GRAFT_STATUS_BAD_LENGTH;
    if (layer == 0 && blockIdx.x == 0 && threadIdx.x == 0) {
        p.status[b] = st;
        p.new_prefix_len[b] = st == 0 ? P + a + 1 : P;
    }
    if (st != 0 || a == 0) return;               // uniform

    // the rows' byte offsets, source and destination; lanes behind the path look up the first page and are not used
    const int32_t* table = block_table + static_cast<size_t>(b) * max_pages;
    auto row_off = [&](int32_t page, int32_t t) {
        return static_cast<u64>(static_cast<int64_t>(page) * p.page_stride +
                                static_cast<int64_t>(t & (GRAFT_PAGE_SIZE - 1)) * p.token_stride) << p.elem_shift;
    };
    u64 src[2], dst[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int32_t k = lane + 1 + 64 * h;
        const int32_t from = k <= a ? P + node[h] : 0, to = k <= a ? P + k : 0;
        const int32_t page_from = table[from / GRAFT_PAGE_SIZE], page_to = table[to / GRAFT_PAGE_SIZE];
        src[h] = row_off(page_from, from);
        dst[h] = row_off(page_to, to);
    }
    // all lanes stay for the copy (their offsets are read across lanes); those behind the last column load it and store nothing
    const int cols = p.Hkv << p.cols_shift;
    const int col = blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = col < cols;
    const int at = live ? col : cols - 1;
    const int g = at >> p.cols_shift;
    const int64_t base = ((static_cast<int64_t>(layer) * p.layer_stride + static_cast<int64_t>(g) * p.head_stride) << p.elem_shift) +
                         static_cast<int64_t>(at - (g << p.cols_shift)) * 16;
    unsigned char* kb = static_cast<unsigned char*>(p.k) + base;
    unsigned char* vb = static_cast<unsigned char*>(p.v) + base;
    auto of_lane = [](u64 v, int l) {
        return (static_cast<u64>(static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(v >> 32), l))) << 32) |
               static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(v), l));
    };
    for (int k0 = 0; k0 < a; k0 += KC_BATCH) {   // row k of the path is number k - 1 here
        const u64 s = k0 < 64 ? src[0] : src[1], d = k0 < 64 ? dst[0] : dst[1];
        Quad kr[KC_BATCH], vr[KC_BATCH];
#pragma unroll
        for (int j = 0; j < KC_BATCH; ++j) {     // (no branch around a load; behind the end the last row is read again)
            const u64 off = of_lane(s, (k0 + j < a ? k0 + j : a - 1) & 63);
            kr[j] = *reinterpret_cast<const Quad*>(kb + off);
            vr[j] = *reinterpret_cast<const Quad*>(vb + off);
        }
#pragma unroll
        for (int j = 0; j < KC_BATCH; ++j) {
            const u64 off = of_lane(d, (k0 + j) & 63);
            if (live && k0 + j < a) {
                *reinterpret_cast<Quad*>(kb + off) = kr[j];
                *reinterpret_cast<Quad*>(vb + off) = vr[j];
            }
        }
    }
}

}  // namespace graft

extern "C" int32_t graft_kv_compact(void* k_cache, void* v_cache, int64_t layer_stride, int32_t n_layers,
                                    int64_t page_stride, int64_t token_stride, int64_t head_stride,
                                    const int32_t* block_table, int32_t max_pages,
                                    const int32_t* prefix_len, const int32_t* path, const int32_t* accept_len,
                                    int32_t B, int32_t depth_cap, int32_t K_max, int32_t Hkv, int32_t D,
                                    int32_t dtype, int32_t* new_prefix_len, int32_t* status, void* stream) {
    using namespace graft;
    if (!k_cache || !v_cache || !block_table || !prefix_len || !path || !accept_len || !new_prefix_len || !status)
        return GRAFT_ERR_NULL;
    if (dtype != GRAFT_F32 && dtype != GRAFT_BF16) return GRAFT_ERR_DTYPE;
    const int32_t es = dtype == GRAFT_F32 ? 4 : 2;
    // 16-byte columns: every stride must keep them aligned
    const int64_t align = 16 / es;
    if (B < 1 || B > 65535 || n_layers < 1 || n_layers > 65535 || depth_cap < 0 || depth_cap >= GRAFT_MAX_NODES ||
        K_max < 1 || K_max > GRAFT_MAX_NODES || Hkv < 1 || Hkv > 65535 || (D != 64 && D != 128) || max_pages < 1 ||
        page_stride < 1 || token_stride < D || head_stride < D || layer_stride < 0 ||
        (n_layers > 1 && layer_stride < 1) || page_stride % align != 0 || token_stride % align != 0 ||
        head_stride % align != 0 || layer_stride % align != 0)
        return GRAFT_ERR_SHAPE;
    if ((reinterpret_cast<size_t>(k_cache) | reinterpret_cast<size_t>(v_cache)) & 15) return GRAFT_ERR_SHAPE;
    // Every workgroup of a sequence reads prefix_len[b] when it starts and one of them writes
    // new_prefix_len[b]: the two arrays must not share memory.
    if (new_prefix_len < prefix_len + B && prefix_len < new_prefix_len + B) return GRAFT_ERR_SHAPE;
    CompactParams p{};
    p.k = k_cache; p.v = v_cache; p.new_prefix_len = new_prefix_len; p.status = status;
    p.layer_stride = layer_stride; p.page_stride = page_stride; p.token_stride = token_stride;
    p.head_stride = head_stride; p.Hkv = Hkv; p.elem_shift = es == 4 ? 2 : 1;
    const int cols_per_head = D * es / 16;       // 8, 16 or 32
    p.cols_shift = __builtin_ctz(static_cast<unsigned>(cols_per_head));
    const int cols = Hkv * cols_per_head;
    const int waves = (cols + 63) / 64;          // per layer and sequence
    const int threads = static_cast<int64_t>(B) * n_layers * waves <= KC_ALONE ? 64 : (64 * waves < KC_THREADS ? 64 * waves : KC_THREADS);
    dim3 grid((cols + threads - 1) / threads, n_layers, B);
    hipLaunchKernelGGL(kv_compact_kernel, grid, dim3(threads), 0, static_cast<hipStream_t>(stream), prefix_len,
                       accept_len, path, block_table, depth_cap, K_max, max_pages, p);
    return check_launch();
}
