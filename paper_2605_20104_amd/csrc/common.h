// Shared host-side helpers of the HIP sources (error bookkeeping, launch checks).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "graft.h"

namespace graft {

// Raw hipError_t of the last failed launch on this thread; defined in api.hip.
void set_last_hip_error(int32_t e);

// Checks the launch that was just enqueued; maps a failure to GRAFT_ERR_HIP.
inline int32_t check_launch() {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_last_hip_error(static_cast<int32_t>(e));
        return GRAFT_ERR_HIP;
    }
    return GRAFT_OK;
}

using u64 = unsigned long long;

// OR of a predicate over a workgroup of two wavefronts (the 128-thread kernels): each wavefront
// puts its ballot's verdict into its own LDS slot, one barrier, everyone reads both slots.  The
// library's __syncthreads_or costs several hundred cycles more, which these launch-latency-bound
// kernels notice.  `slots` is LDS, two words, not used for anything else until the next barrier;
// the barrier also orders every LDS write made before the call.
__device__ __forceinline__ bool workgroup_or_128(bool pred, int32_t* slots) {
    const bool wave_any = __builtin_amdgcn_ballot_w64(pred) != 0;
    if ((threadIdx.x & 63) == 0) slots[threadIdx.x >> 6] = wave_any ? 1 : 0;
    __syncthreads();
    return (slots[0] | slots[1]) != 0;
}

// v from the lane that the DPP control names (0xB1: lane ^ 1, 0x4E: lane ^ 2, 0x141: mirror
// within 8 lanes, 0x140: mirror within 16 lanes), both halves of the 64-bit value.
template <int DPP_CTRL>
__device__ __forceinline__ u64 dpp_u64(u64 v) {
    const int lo = static_cast<int>(static_cast<unsigned>(v)), hi = static_cast<int>(static_cast<unsigned>(v >> 32));
    const unsigned lo2 = static_cast<unsigned>(__builtin_amdgcn_update_dpp(lo, lo, DPP_CTRL, 0xf, 0xf, false));
    const unsigned hi2 = static_cast<unsigned>(__builtin_amdgcn_update_dpp(hi, hi, DPP_CTRL, 0xf, 0xf, false));
    return (static_cast<u64>(hi2) << 32) | lo2;
}

// Maximum of a 64-bit key over one 64-lane wavefront (all lanes get it).  Four DPP steps
// reduce each row of 16 lanes (register-to-register, no LDS crossbar); the gfx950 lane
// swaps then combine the rows: permlane16_swap(x, x) returns {rows 0,0,2,2} and
// {rows 1,1,3,3} of x, permlane32_swap(x, x) returns {low half twice} and {high half twice}.
__device__ __forceinline__ u64 wave_max_u64(u64 v) {
    u64 o;
    o = dpp_u64<0xB1>(v);  v = o > v ? o : v;
    o = dpp_u64<0x4E>(v);  v = o > v ? o : v;
    o = dpp_u64<0x141>(v); v = o > v ? o : v;
    o = dpp_u64<0x140>(v); v = o > v ? o : v;
    {
        const unsigned lo = static_cast<unsigned>(v), hi = static_cast<unsigned>(v >> 32);
        const auto rl = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto rh = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        const u64 a = (static_cast<u64>(rh[0]) << 32) | rl[0], b = (static_cast<u64>(rh[1]) << 32) | rl[1];
        v = a > b ? a : b;
    }
    {
        const unsigned lo = static_cast<unsigned>(v), hi = static_cast<unsigned>(v >> 32);
        const auto rl = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto rh = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        const u64 a = (static_cast<u64>(rh[0]) << 32) | rl[0], b = (static_cast<u64>(rh[1]) << 32) | rl[1];
        v = a > b ? a : b;
    }
    return v;
}

// Maximum of a float over one 64-lane wavefront (all lanes get it); same steps as above.
template <int DPP_CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
    const int b = __float_as_int(v);
    return __int_as_float(__builtin_amdgcn_update_dpp(b, b, DPP_CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float wave_max_f32(float v) {
    v = __builtin_fmaxf(v, dpp_f32<0xB1>(v));
    v = __builtin_fmaxf(v, dpp_f32<0x4E>(v));
    v = __builtin_fmaxf(v, dpp_f32<0x141>(v));
    v = __builtin_fmaxf(v, dpp_f32<0x140>(v));
    {
        const unsigned u = __float_as_uint(v);
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        v = __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    {
        const unsigned u = __float_as_uint(v);
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        v = __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    return v;
}

// Maximum of a 32-bit number over one 64-lane wavefront (all lanes get it); same steps again.
template <int DPP_CTRL>
__device__ __forceinline__ unsigned max_dpp_u32(unsigned v) {
    const unsigned o = static_cast<unsigned>(__builtin_amdgcn_update_dpp(static_cast<int>(v), static_cast<int>(v), DPP_CTRL, 0xf, 0xf, false));
    return o > v ? o : v;
}
__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
    v = max_dpp_u32<0xB1>(v);
    v = max_dpp_u32<0x4E>(v);
    v = max_dpp_u32<0x141>(v);
    v = max_dpp_u32<0x140>(v);
    {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = r[0] > r[1] ? r[0] : r[1];
    }
    {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = r[0] > r[1] ? r[0] : r[1];
    }
    return v;
}

// wave_max_u64 for keys whose upper words hardly ever agree: their maximum decides (one instruction a step
// instead of five), the lower words are compared only where several lanes have it.  In the matrix refresh, which takes
// k of them per chunk and per row, us a call in a graph: 8 x 96 rows of 32000 logits 50.3 -> 48.1, 8 x 24 18.6 -> 18.0.
__device__ __forceinline__ u64 wave_max_key(u64 v) {
    const unsigned hi = static_cast<unsigned>(v >> 32), lo = static_cast<unsigned>(v);
    const unsigned top = wave_max_u32(hi);
    const u64 at = __builtin_amdgcn_ballot_w64(hi == top);           // never empty
    unsigned low;
    if ((at & (at - 1)) == 0)                                        // uniform
        low = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(lo), __builtin_ctzll(at)));
    else
        low = wave_max_u32(hi == top ? lo : 0u);
    return (static_cast<u64>(top) << 32) | low;
}

// What a wavefront's lanes have written to LDS is what its lanes read from here on, and the other way round.  (A wavefront's
// LDS operations complete in order; this keeps the compiler from changing that order.)
__device__ __forceinline__ void wavefront_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Maximum over the four lanes l, l + 16, l + 32, l + 48 (the four 16-lane rows of a wavefront),
// all four get it: the two lane swaps of gfx950, no trip through the LDS crossbar.
__device__ __forceinline__ float rows_max_f32(float v) {
    {
        const unsigned u = __float_as_uint(v);
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        v = __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    {
        const unsigned u = __float_as_uint(v);
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        v = __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    return v;
}

// Sixteen bytes of logits, ONCE: with a load that says that they are not needed again.  Where the rows are more than the
// 256 MB Infinity Cache still holds behind whoever wrote them, that is faster: acceptance of 8 x 48 rows of 151936 (233 MB), written in
// front of it, 55.7 -> 49.7 us, 16 x 64 of 60001 (246 MB) 59.2 -> 49.7, matrix refresh of 16 x 128 of 128256 178.5 -> 165.5.  Below it is
// slower where they have just been written: 80 MB 19.6 / 20.5, 100 MB 22.4 / 23.6, 184 MB 35.5 / 35.2, 210 MB 42.9 / 43.8.
template <bool ONCE> __device__ __forceinline__ float4 load_logits(const float4* p) {
    if constexpr (!ONCE) return *p;
    typedef float float4_t __attribute__((ext_vector_type(4)));
    const float4_t x = __builtin_nontemporal_load(reinterpret_cast<const float4_t*>(p));
    return float4{x[0], x[1], x[2], x[3]};
}
inline bool read_once(int64_t rows, int32_t V) { return rows * V * 4 > (int64_t{208} << 20); }

// A logits row cut for 16-byte loads whatever its length and address: `head` elements up to the first
// 16-byte boundary, `quads` aligned groups of four, `tail` elements behind them.  The groups are dealt to
// `chunks` workgroups, `per` to each, the edges (at most three elements each) go to the first and the
// last of them, one element per thread.  Rows of an odd length used to be read
// element by element: 8 x 48 rows of 151937 took 84 us in the acceptance, 46 now, as rows of 151936 do;
// 8 x 64 rows of 50257 took 86 us in the matrix refresh, 40 then (logits from memory, not from a cache).
struct RowChunk {
    const float4* quad;      // aligned
    int32_t head, q0, q1;    // this workgroup's groups; group q starts at element head + 4 q
    int32_t edge;            // number of edge elements of this workgroup (threads 0 .. edge - 1), at most six
    int32_t edge_head, behind;
    __device__ __forceinline__ int32_t edge_at(int32_t t) const { return t < edge_head ? t : behind + t - edge_head; }
};
constexpr int ROW_EDGES = 6;
__device__ __forceinline__ RowChunk row_chunk(const float* row, int32_t V, int chunk, int chunks, int32_t per) {
    const int32_t to_boundary = static_cast<int32_t>((16 - (reinterpret_cast<size_t>(row) & 15)) & 15) / 4;
    RowChunk c;
    c.head = to_boundary < V ? to_boundary : V;
    const int32_t quads = (V - c.head) / 4;
    c.quad = reinterpret_cast<const float4*>(row + c.head);
    c.q0 = chunk * per < quads ? chunk * per : quads;
    c.q1 = c.q0 + per < quads ? c.q0 + per : quads;
    c.behind = c.head + 4 * quads;
    c.edge_head = chunk == 0 ? c.head : 0;
    c.edge = c.edge_head + (chunk == chunks - 1 ? V - c.behind : 0);
    return c;
}

// Workgroups per row of a scan of `rows` rows, and groups per workgroup.  A workgroup of the scans costs the same set-up and
// selection whatever it holds, so a row goes to as few as take ROW_QUADS groups each (every row went to
// GRAFT_ARGMAX_CHUNKS), but to as many as it takes to give the chip ROW_FILL workgroups where the rows are few.
// us a call in a graph, matrix refresh with k = 8 / acceptance, 16 workgroups a row -> this rule:
//   16 x 128 rows of 8000 111.4 -> 22.0 / 43.5 -> 16.0    8 x 96 rows of 32000 52.4 -> 27.2 / 23.1 -> 22.3
//   8 x 24 rows of 32000 19.7 -> 14.3 / 10.4 -> 9.8       16 x 64 rows of 60001 73.0 -> 50.3 / 45.6 -> 44.9
//   1 x 40 rows of 128256, 8 x 48 of 151936 and 16 x 128 of 128256 (16 workgroups a row either way) as before.
// ROW_QUADS: all 12 loads of a thread in use (3072) make the refresh of 16 x 128 rows of 128256 180 us instead of 170
// (11 workgroups a row; they select while nobody loads), 1536 groups that of 16 x 64 rows of 32000 36.4 instead of 32.1.
// ROW_FILL: with 2048 and 4096 the refresh of 8 x 24 rows of 32000 takes 16.9 and 19.2 us, with 1024 14.3.
// The rows of absent nodes count although their workgroups leave at once: the host does not know n_nodes.  So the rule is made for
// slots that are in use, and 16 workgroups a row are faster where hardly any are; rows of 32000, 16 a row / this rule:
// refresh of 4 x 64 slots, 1, 4, 8, 24, 64 nodes each: 10.0 / 11.4, 10.4 / 11.8, 12.6 / 12.0, 14.9 / 12.0, 22.9 / 13.8 us; acceptance
// of 8 x 64: 8.5 / 9.1, 8.8 / 9.5, 9.5 / 9.6, 12.8 / 9.7, 20.9 / 14.6.  Of 16 x 128 slots with 8 nodes, rows of 8000: 24.1 / 15.3
// and 15.0 / 9.6.
constexpr int32_t ROW_QUADS = 8 * 256;
constexpr int64_t ROW_FILL = 1024;
struct RowCut { int32_t chunks, per; };
inline RowCut row_cut(int64_t rows, int32_t V) {
    const int32_t quads = V / 4;
    int64_t chunks = (quads + ROW_QUADS - 1) / ROW_QUADS;
    const int64_t fill = (ROW_FILL + rows - 1) / rows;
    if (chunks < fill) chunks = fill;
    if (chunks > GRAFT_ARGMAX_CHUNKS) chunks = GRAFT_ARGMAX_CHUNKS;
    return {static_cast<int32_t>(chunks), static_cast<int32_t>((quads + chunks - 1) / chunks)};
}

}  // namespace graft
