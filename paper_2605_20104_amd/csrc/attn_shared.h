// What the attention translation units share: kernel parameters, launch plans, launch helpers.
#pragma once
#include <hip/hip_ext.h>

#include "common.h"

namespace graft {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));

struct AttnParams {
    const void* q;
    const void* k;
    const void* v;
    void* out;
    const int32_t* block_table;
    const int32_t* prefix_len;
    const int32_t* n_nodes;
    const u64* mask;
    // partial rows of the splits.  MFMA path: fp16 [B][Hkv][splits][R_pad/16][D/32] blocks of 1 KB: [lane][2][4],
    // lane = MFMA accumulator lane, two adjacent 16-dim tiles per block; with 32-row blocks [R_pad/32][D/16] of [lane][8]; direct path: fp32 [B][Hkv][splits][R_pad][D]
    unsigned short* ws_o;
    // MFMA path: [B][Hkv][splits][R_pad][4] (reference in log2 units, sum, scale of the stored row, 0; with 32-row blocks a
    // scale for either half of the dims); direct path:
    // [B][Hkv][splits][R_pad][2] (max in log2 units, sum)
    float* ws_ml;
    int64_t page_stride, token_stride, head_stride;
    int32_t max_pages, B, K_max, Hq, Hkv, G, R, R_pad, n_splits, n_row_tiles;
    int32_t g_magic;    // ceil(2^16 / G): r / G == (r * g_magic) >> 16 for r < 4096, G <= 16
    float scale_log2e;  // softmax scale * log2(e)
    unsigned long long* stamps;   // timing build: AT_STAMPS values per workgroup, or null (always null otherwise)
};

// Division by a number that the host knows: x / d == (x * magic31(d)) >> 31 for x >= 0, d >= 1 with x (d - 1) < 2^31 (m d - 2^31 is
// at most d - 1, so x m / 2^31 is past x / d by at most x (d - 1) / (2^31 d), which must stay below 1 / d).  A division is some
// thirty dependent instructions, and several stand in front of a workgroup's first requests.
inline uint32_t magic31(uint32_t d) { return ((1u << 31) + d - 1u) / d; }
__host__ __device__ __forceinline__ int div31(int x, uint32_t magic) {
    return static_cast<int>((static_cast<u64>(static_cast<unsigned>(x)) * magic) >> 31);
}
// The same for 0 <= x < 2^31 and any d: 2^shift, the least power of two from d on, leaves the multiplier 31 bits and more.
struct Magic { uint32_t m; int32_t shift; };
inline Magic magic_any(uint32_t d) {
    int32_t shift = 0;
    while ((u64{1} << shift) < d) ++shift;
    return {static_cast<uint32_t>(((u64{1} << (31 + shift)) + d - 1) / d), shift};
}
__host__ __device__ __forceinline__ int div_any(int x, uint32_t magic, int shift) {
    return static_cast<int>((static_cast<u64>(static_cast<unsigned>(x)) * magic) >> (31 + shift));
}
// x / d for x, d < 2^24, by a number that has no such bound.
__device__ __forceinline__ int div24(int x, int d) {
    return static_cast<int>((static_cast<unsigned>(x) & 0xffffffu) / (static_cast<unsigned>(d) & 0xffffffu));
}
// Workgroups go to the 8 XCDs (each with its own L2 and its own compute units) round-robin by their
// linear index.  The row tiles of a unit, one (sequence, KV head, split), read the same keys and
// values: they get the same XCD and neighbouring slots on it, so that all but the first reader find
// them in that XCD's L2.  Units are dealt round-robin, eight at a time; the row tiles of what is left
// over are dealt one by one, so that the XCDs' shares differ by one workgroup at most (with whole
// units only, 50 units of 5 tiles put 35 workgroups on two XCDs of 32 compute units: a second round
// for a job that was planned to fill the chip once, 71 us instead of 42).
struct WorkItem { int unit, row_tile; };                         // unit < 0: padding of the grid
inline unsigned xcd_grid(int64_t n_units, int64_t n_row_tiles) {
    return static_cast<unsigned>(8 * ((n_units / 8) * n_row_tiles + (n_units % 8 * n_row_tiles + 7) / 8));
}
__device__ __forceinline__ WorkItem xcd_work_item(int n_units, int n_row_tiles, uint32_t row_tiles_magic) {
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int whole = (n_units >> 3) * n_row_tiles;               // slots of an XCD that take whole units
    const bool left = slot >= whole;
    const int s = left ? (slot - whole) * 8 + xcd : slot;
    const int u = div31(s, row_tiles_magic), t = s - u * n_row_tiles;
    const int unit = left ? (n_units & ~7) + u : u * 8 + xcd;
    return {unit < n_units ? unit : -1, t};
}

// Compute units of the current device (256 when it cannot be asked, e.g. without a GPU).
int device_compute_units();

// The direct path (tree_attn_direct.hip): launch shape and launch.
struct DirectPlan {
    int mb, rg, n_row_tiles, n_splits, r_pad;
    size_t ws_o_bytes, ws_bytes;
    double cost;        // estimated cycles
    bool parts;         // fp32 on the 16-bit matrix cores (tree_attn_parts.hip)
};
DirectPlan plan_direct(int32_t B, int32_t K_max, int32_t Hq, int32_t Hkv, int32_t D, int32_t max_pages, int32_t dtype,
                       bool may_split);
int32_t launch_parts(const DirectPlan& pl, const AttnParams& p, int32_t D, hipStream_t s);
int32_t launch_direct(const DirectPlan& pl, AttnParams p, int32_t D, int32_t dtype, void* workspace, hipStream_t s);

// Profiling hook state (per host thread): event pairs attached to the main kernel's dispatch
// (hipExtLaunchKernelGGL: the events then carry the kernel's own begin and end time stamps,
// without the dispatch latency that events recorded around a launch would include).
struct ProfileHook {
    hipEvent_t* start = nullptr;
    hipEvent_t* stop = nullptr;
    int32_t n = 0, i = 0;
};
extern thread_local ProfileHook g_prof;

template <class Kernel, class... Args>
static void launch_main(Kernel kernel, dim3 grid, dim3 block, unsigned lds_bytes, hipStream_t s, Args... args) {
    if (g_prof.i < g_prof.n) {
        hipExtLaunchKernelGGL(kernel, grid, block, lds_bytes, s, g_prof.start[g_prof.i], g_prof.stop[g_prof.i], 0, args...);
        ++g_prof.i;
    } else {
        hipLaunchKernelGGL(kernel, grid, block, lds_bytes, s, args...);
    }
}

// The main kernels' first arguments arrive in scalar registers (the build's kernarg preload) where the rest is a trip to
// memory: they are what a workgroup needs to find its sequence and to request its lengths.  n_splits <= 64, row tiles <= 128
// and, from the limit on a launch's work-items, fewer than 2^24 workgroups, as div31 wants it.
#define GRAFT_ATTN_ARGS                                                                                                        \
    const int32_t *n_nodes, const int32_t *prefix_len, int32_t n_units, int32_t n_row_tiles, uint32_t row_tiles_magic, int32_t n_splits, \
        uint32_t splits_magic, int32_t n_kv_heads, int32_t row_groups, uint32_t row_groups_magic, int32_t key_groups,                \
        uint32_t key_groups_magic, AttnParams p
template <class Kernel>
static void launch_attn(Kernel kernel, dim3 grid, dim3 block, unsigned lds_bytes, hipStream_t s, const AttnParams& p, int32_t row_groups,
                        int32_t key_groups) {
    launch_main(kernel, grid, block, lds_bytes, s, p.n_nodes, p.prefix_len, p.B * p.Hkv * p.n_splits, p.n_row_tiles,
                magic31(static_cast<uint32_t>(p.n_row_tiles)), p.n_splits, magic31(static_cast<uint32_t>(p.n_splits)), p.Hkv, row_groups,
                magic31(static_cast<uint32_t>(row_groups)), key_groups, magic31(static_cast<uint32_t>(key_groups)), p);
}

// The rest of AttnParams that the set-up reads, requested at once at the top of the kernel.  Left to itself the compiler
// loads each argument where it is first used, and in a chain of dependent trips (lengths, page table, first keys) every
// such load is a trip of its own.
__device__ __forceinline__ void await_setup_args(const AttnParams& p) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" : : "s"(p.q), "s"(p.k), "s"(p.v), "s"(p.block_table), "s"(p.mask), "s"(p.page_stride), "s"(p.token_stride),
                 "s"(p.head_stride), "s"(p.max_pages), "s"(p.K_max), "s"(p.Hq), "s"(p.G), "s"(p.R), "s"(p.g_magic), "s"(p.scale_log2e));
}

// A wavefront-uniform value that the compiler takes for one that differs between lanes: what is loaded with it stays in
// a vector register until it is asked for, instead of being waited for and moved to a scalar register on the spot.
__device__ __forceinline__ int per_lane(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Which of the 32 tokens from tree slot s on (s = token - prefix length, negative inside the prefix) a
// row sees, as bits: all of the prefix, of the first n tree slots those in the row's ancestor mask.  word(k)
// returns the mask's 32-bit word k, 0 <= k < 4.  s and n are wavefront-uniform, so that the words are
// picked by scalar conditions and a row costs one funnel shift and one AND.
template <class Word>
__device__ __forceinline__ unsigned visible_window(int s, int n, Word&& word) {
    const int w = s >> 5, left = n - s;
    const unsigned lo = w < 0 ? ~0u : (w < 4 ? word(w) : 0u);
    const unsigned hi = w < -1 ? ~0u : (w < 3 ? word(w + 1) : 0u);
    const unsigned slots = left >= 32 ? ~0u : (left <= 0 ? 0u : (1u << left) - 1u);
    return __builtin_amdgcn_alignbit(hi, lo, static_cast<unsigned>(s) & 31u) & slots;
}
// x where bit `bit` of the window is set, -inf elsewhere: a bit-field extract and a bit select.
__device__ __forceinline__ float keep_visible(float x, unsigned window, int bit) {
    const unsigned m = static_cast<unsigned>(__builtin_amdgcn_sbfe(static_cast<int>(window), bit, 1));
    return __uint_as_float((__float_as_uint(x) & m) | (0xff800000u & ~m));
}

// Loads of a merge, through a buffer descriptor: zeros, without a trip to memory, where the offset lies behind its end.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t merge_buffer(const void* base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, static_cast<int>(bytes), 0x00020000);
}
// Two fp32 -> one packed pair of bf16 (round to nearest even): v_cvt_pk_bf16_f32.
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{lo, hi}, bf16x2));
}

}  // namespace graft
