// What the direct path's two kernels share: size of a workgroup, row sums, the merge of key groups through LDS.
#pragma once
#include "attn_shared.h"

namespace graft {

constexpr int DR_WAVES = 8;                     // wavefronts per workgroup, two per SIMD
constexpr int DR_THREADS = 64 * DR_WAVES;
constexpr float DR_LAZY_LOG2 = 16.0f;           // a row keeps its reference while exponents stay below 16
constexpr int DR_MAX_SPLITS = 32;
constexpr int DR_MASK_BYTES = 2048;             // ancestor masks of a sequence
constexpr int DR_LDS_BYTES = 160 * 1024;

__device__ __forceinline__ unsigned lds_offset(const void* p) {
    return static_cast<unsigned>(reinterpret_cast<size_t>((const __attribute__((address_space(3))) unsigned char*)(p)));
}

// Sum / maximum over the lanes that hold the same row: lane, lane + 32 and, with 16 rows to a block, those 16 apart.
template <int RB> __device__ __forceinline__ float row_sum(float v) {
    if constexpr (RB == 16) {
        const unsigned u = __float_as_uint(v);
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int RB> __device__ __forceinline__ float row_max(float v) {
    if constexpr (RB == 16) return rows_max_f32(v);
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Workgroup barrier that orders LDS traffic only: keys and values on their way stay in flight.
__device__ __forceinline__ void lds_only_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ void store4(float* p, const floatx4& v) { *reinterpret_cast<floatx4*>(p) = v; }
__device__ __forceinline__ void store4(__bf16* p, const floatx4& v) {
    *reinterpret_cast<uintx2*>(p) = uintx2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
}

// Merge of a workgroup's key groups behind the loop: [group][rows][D + 4] partial rows and [group][rows] (m, l) in LDS.  All reads of
// a piece in flight: one after the other they took 1 us.  row0: the workgroup's first row; part: of its partial rows.
template <typename T, int D, int KG>
__device__ __forceinline__ void merge_key_groups(const AttnParams& p, const float* merge_lds, const float* ml_lds, int rows, int row0, int tid,
                                                 int b, int g, int n, int n_splits, size_t part) {
    constexpr int PITCH = D + 4;
    float* ws_o = reinterpret_cast<float*>(p.ws_o);
    for (int x = tid; x < rows * (D / 4); x += DR_THREADS) {
        const int lr = x / (D / 4), d4 = x % (D / 4);
        float2 ml[KG];
        floatx4 part_o[KG];
#pragma unroll
        for (int k = 0; k < KG; ++k) ml[k] = *reinterpret_cast<const float2*>(ml_lds + 2 * (k * rows + lr));
#pragma unroll
        for (int k = 0; k < KG; ++k) part_o[k] = *reinterpret_cast<const floatx4*>(merge_lds + (k * rows + lr) * PITCH + 4 * d4);
        float mm = -INFINITY;
#pragma unroll
        for (int k = 0; k < KG; ++k) mm = fmaxf(mm, ml[k].x);
        float den = 0.f;
        floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KG; ++k) {
            const float f = ml[k].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[k].x - mm);
            den += f * ml[k].y;
            acc += part_o[k] * f;
        }
        const int r = row0 + lr;
        if (n_splits == 1) {
            if (r < p.R) {
                const int i = (r * p.g_magic) >> 16;
                const bool keep = i < n && den > 0.f;
                const floatx4 y = keep ? acc * (1.0f / den) : floatx4{0.f, 0.f, 0.f, 0.f};
                store4(static_cast<T*>(p.out) + ((static_cast<size_t>(b) * p.K_max + i) * p.Hq + g * p.G + (r - i * p.G)) * D + 4 * d4, y);
            }
        } else {
            store4(ws_o + (part + r) * D + 4 * d4, acc);
            if (d4 == 0) {
                p.ws_ml[2 * (part + r)] = mm;
                p.ws_ml[2 * (part + r) + 1] = den;
            }
        }
    }
}

// Launch of a main kernel of the direct path.
template <typename T, int D, auto KERNEL>
int32_t launch_pieces(const DirectPlan& pl, const AttnParams& p, unsigned lds, hipStream_t s) {
    if (lds > 65536) {                                            // more than the default limit needs opting in, once per device
        static thread_local int done_device = -1;
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) dev = 0;
        if (done_device != dev) {
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, DR_LDS_BYTES);
            done_device = dev;
        }
    }
    // A launch holds fewer than 2^32 work-items.  Batches that need more go in pieces of whole sequences: one
    // sequence has at most 65535 * 128 workgroups (KV heads, row tiles), which fits.
    constexpr int64_t max_workgroups = ((int64_t{1} << 32) - 1) / DR_THREADS - 8;
    const int64_t per_sequence = static_cast<int64_t>(p.Hkv) * pl.n_splits * pl.n_row_tiles;
    const int64_t piece = max_workgroups / per_sequence;
    AttnParams part = p;
    for (int64_t b = 0; b < p.B; b += piece) {
        part.B = static_cast<int32_t>(p.B - b < piece ? p.B - b : piece);
        const size_t elements = static_cast<size_t>(b) * p.K_max * p.Hq * D;
        part.q = static_cast<const T*>(p.q) + elements;
        part.out = static_cast<T*>(p.out) + elements;
        part.block_table = p.block_table + b * p.max_pages;
        part.prefix_len = p.prefix_len + b;
        part.n_nodes = p.n_nodes + b;
        part.mask = p.mask + b * p.K_max * GRAFT_MASK_WORDS;
        launch_attn(KERNEL, dim3(xcd_grid(static_cast<int64_t>(part.B) * p.Hkv * pl.n_splits, pl.n_row_tiles)), dim3(DR_THREADS), lds, s,
                    part, pl.rg, DR_WAVES / pl.rg);
        const int32_t rc = check_launch();
        if (rc != GRAFT_OK) return rc;
    }
    return GRAFT_OK;
}

}  // namespace graft
