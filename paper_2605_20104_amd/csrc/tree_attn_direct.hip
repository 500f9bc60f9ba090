// graft_tree_attn, direct path: fp32 storage (any head size) and bf16 with D = 64.
//
// Keys and values go from memory straight into registers, in the layout the matrix
// instructions take them in; no LDS staging and no barrier inside the loop.  That is possible
// because a wavefront owns its keys: the wavefronts of a workgroup split a key range between
// them (kg key groups), as well as the query rows (rg row groups of MB 16-row blocks), and
// merge at the end through LDS, so that a short prefix is spread over the chip with few or no
// partial results in memory.
//   fp32 : v_mfma_f32_16x16x4_f32 (full fp32 products and sums, 32 cycles each).  The kernel is
//          bound by them: 64 (D = 128) or 32 (D = 64) per 16 keys and 16 rows.
//   bf16 : v_mfma_f32_16x16x32_bf16 on raw Q and K (exact products, fp32 sums); the softmax scale
//          is applied in fp32, and probabilities enter the second product as the sum of two bf16
//          numbers (relative error 2^-17: far below the rounding of the result).  Bound by the
//          vector ALUs (exp2 and the packing of probabilities).
// Operand layouts (lane = 16 lg + l16).  First product: S^T = K Q^T, A = K (key l16), B = Q^T
// (row l16), so a lane gets 4 keys (4 lg + i) of one row, and these are the B operand of the
// second product O^T = V^T P^T without any exchange between lanes: its contraction index runs
// over the same keys (16 c + 4 lg + i).  Its A operand wants, per lane, one dim of those keys: the
// assignment of dims to the MFMA's 16 rows is free, so a lane loads a row piece of D/16 (fp32: 4)
// consecutive dims per key with one wide load and uses one of them per MFMA; bf16 pairs of keys
// are interleaved with v_perm_b32.
//
// Latency: lengths -> page table -> first keys are three dependent trips; Q and the ancestor
// masks travel with the lengths.  The table entries of a wavefront's tiles sit in one vector
// register (lane = tile and page), one trip for 32 (fp32: 64) tiles.  The next tile's keys and
// values are requested before the current tile is computed.
#include <type_traits>

#include "attn_shared.h"

namespace graft {

constexpr int DR_WAVES = 8;                     // wavefronts per workgroup, two per SIMD
constexpr int DR_THREADS = 64 * DR_WAVES;
constexpr float DR_LAZY_LOG2 = 16.0f;           // a row keeps its reference while exponents stay below 2^16
constexpr int DR_MAX_SPLITS = 32;

__device__ __forceinline__ float rows_sum_f32(float v) {
    {
        const unsigned u = __float_as_uint(v);
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    {
        const unsigned u = __float_as_uint(v);
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    return v;
}

// Per storage type: keys per tile, registers of a tile's keys and values, the two products.
template <typename T, int D> struct DirectOps;

template <int D> struct DirectOps<float, D> {
    static constexpr int TK = 16;               // keys per tile
    static constexpr int NO = D / 16;           // floatx4 accumulators per row block
    static constexpr int NC = 1;                // score tiles of 16 keys
    struct Q { floatx4 v[D / 16]; };
    struct K { floatx4 r[D / 16]; };
    struct V { floatx4 r[4][D / 64]; };
    static __device__ __forceinline__ void load_q(Q& q, const float* row, int lg) {
#pragma unroll
        for (int s = 0; s < D / 16; ++s) q.v[s] = *reinterpret_cast<const floatx4*>(row + 16 * s + 4 * lg);
    }
    // a lane's byte offset inside its key's row, for K and for V
    static __device__ __forceinline__ unsigned k_lane(int lg) { return 16 * lg; }
    static __device__ __forceinline__ unsigned v_lane(int l16) { return 16 * l16; }
    static __device__ __forceinline__ void load_k(K& t, int, const char* base, unsigned off) {
#pragma unroll
        for (int s = 0; s < D / 16; ++s) t.r[s] = *reinterpret_cast<const floatx4*>(base + off + 64 * s);
    }
    // values of key i (of this lane's four)
    static __device__ __forceinline__ void load_v(V& t, int, int i, const char* base, unsigned off) {
#pragma unroll
        for (int h = 0; h < D / 64; ++h) t.r[i][h] = *reinterpret_cast<const floatx4*>(base + off + 256 * h);
    }
    static __device__ __forceinline__ void scores(const K& t, const Q& q, floatx4 (&s)[NC]) {
        s[0] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int d = 0; d < D / 16; ++d)
#pragma unroll
            for (int j = 0; j < 4; ++j) s[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.r[d][j], q.v[d][j], s[0], 0, 0, 0);
    }
    static constexpr bool SUM_MFMA = false;
    static constexpr bool FREES_V = false;      // accumulate() still reads the loaded values
    struct A {};
    static __device__ __forceinline__ void arrange(const V&, A&) {}
    static __device__ __forceinline__ void accumulate(const V& t, const A&, const floatx4 (&p)[NC], floatx4 (&o)[NO], floatx4&) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < D / 64; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    o[4 * h + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.r[i][h][j], p[0][i], o[4 * h + j], 0, 0, 0);
    }
    // the four consecutive dims starting at dim(u, lg), u < D/16
    static __device__ __forceinline__ int dim(int u, int lg) { return 64 * (u >> 2) + 16 * lg + 4 * (u & 3); }
    static __device__ __forceinline__ floatx4 piece(const floatx4 (&o)[NO], int u) {
        const int h = u >> 2, i = u & 3;
        return floatx4{o[4 * h][i], o[4 * h + 1][i], o[4 * h + 2][i], o[4 * h + 3][i]};
    }
};

template <int D> struct DirectOps<__bf16, D> {
    static constexpr int TK = 32;
    static constexpr int NO = D / 16;
    static constexpr int NC = 2;
    static constexpr int W = D / 32;            // 32-bit words of a lane's row piece (D/16 dims)
    struct Q { bf16x8 v[D / 32]; };
    struct K { bf16x8 r[2][D / 32]; };
    struct V { unsigned r[8][W]; };
    static __device__ __forceinline__ void load_q(Q& q, const __bf16* row, int lg) {
#pragma unroll
        for (int s = 0; s < D / 32; ++s) q.v[s] = *reinterpret_cast<const bf16x8*>(row + 32 * s + 8 * lg);
    }
    static __device__ __forceinline__ unsigned k_lane(int lg) { return 16 * lg; }
    static __device__ __forceinline__ unsigned v_lane(int l16) { return 4 * W * l16; }
    static __device__ __forceinline__ void load_k(K& t, int c, const char* base, unsigned off) {
#pragma unroll
        for (int s = 0; s < D / 32; ++s) t.r[c][s] = *reinterpret_cast<const bf16x8*>(base + off + 64 * s);
    }
    static __device__ __forceinline__ void load_v(V& t, int c, int i, const char* base, unsigned off) {
        if constexpr (W == 2) {
            const uintx2 x = *reinterpret_cast<const uintx2*>(base + off);
            t.r[4 * c + i][0] = x[0];
            t.r[4 * c + i][1] = x[1];
        } else {
            const uintx4 x = *reinterpret_cast<const uintx4*>(base + off);
#pragma unroll
            for (int w = 0; w < W; ++w) t.r[4 * c + i][w] = x[w];
        }
    }
    static __device__ __forceinline__ void scores(const K& t, const Q& q, floatx4 (&s)[NC]) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            s[c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int d = 0; d < D / 32; ++d) s[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t.r[c][d], q.v[d], s[c], 0, 0, 0);
        }
    }
    // V^T operands: one dim, eight keys per lane
    static constexpr bool SUM_MFMA = true;      // row sums through the matrix cores, which have time left here
    static constexpr bool FREES_V = true;       // arrange() copies: the next values can be requested after it
    struct A { uintx4 a[NO]; };
    static __device__ __forceinline__ void arrange(const V& t, A& v) {
#pragma unroll
        for (int w = 0; w < W; ++w)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v.a[2 * w][j] = __builtin_amdgcn_perm(t.r[2 * j + 1][w], t.r[2 * j][w], 0x05040100u);
                v.a[2 * w + 1][j] = __builtin_amdgcn_perm(t.r[2 * j + 1][w], t.r[2 * j][w], 0x07060302u);
            }
    }
    static __device__ __forceinline__ void accumulate(const V&, const A& v, const floatx4 (&p)[NC], floatx4 (&o)[NO], floatx4& sum) {
        uintx4 hi, lo;                          // p = hi + lo, both bf16 (hi: truncated, so p - hi is exact)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float p0 = p[j >> 1][2 * (j & 1)], p1 = p[j >> 1][2 * (j & 1) + 1];
            const unsigned b0 = __float_as_uint(p0), b1 = __float_as_uint(p1);
            hi[j] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
            lo[j] = pack_bf16(p0 - __uint_as_float(b0 & 0xffff0000u), p1 - __uint_as_float(b1 & 0xffff0000u));
        }
        const bf16x8 ph = __builtin_bit_cast(bf16x8, hi), pl = __builtin_bit_cast(bf16x8, lo);
        const bf16x8 ones = __builtin_bit_cast(bf16x8, uintx4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
        sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, ph, sum, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < NO; ++e) {
            const bf16x8 a = __builtin_bit_cast(bf16x8, v.a[e]);
            o[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, ph, o[e], 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < NO; ++e) {
            const bf16x8 a = __builtin_bit_cast(bf16x8, v.a[e]);
            o[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, pl, o[e], 0, 0, 0);
        }
        sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pl, sum, 0, 0, 0);
    }
    // dims (4 lg + i) * D/16 + e: D/4 consecutive dims per lane
    static __device__ __forceinline__ int dim(int u, int lg) { return lg * (D / 4) + 4 * u; }
    static __device__ __forceinline__ floatx4 piece(const floatx4 (&o)[NO], int u) {
        floatx4 r;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int f = 4 * u + x;
            r[x] = o[f % NO][f / NO];
        }
        return r;
    }
};

__device__ __forceinline__ void store4(float* p, const floatx4& v) { *reinterpret_cast<floatx4*>(p) = v; }
__device__ __forceinline__ void store4(__bf16* p, const floatx4& v) {
    *reinterpret_cast<uintx2*>(p) = uintx2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
}

// p.R_pad = rows covered by the row tiles; rg (row groups) and the rest of the shape as below
template <typename T, int D, int MB>
__global__ __launch_bounds__(DR_THREADS, 2) void tree_attn_direct_kernel(AttnParams p, int32_t rg) {
    using Ops = DirectOps<T, D>;
    constexpr int TK = Ops::TK, NO = Ops::NO, NC = Ops::NC;
    // the next tile in registers of its own while the current one is computed, where they suffice
    constexpr bool DOUBLE = MB * D <= 128;
    constexpr bool MASK_HELD = MB <= 2;         // the rows' ancestor masks in registers, else in LDS
    constexpr int PITCH = D + 4;                // LDS row pitch of the merge: 16 rows at consecutive 16-byte slots
    // with more than one key group [wave][16 MB][PITCH], then (m, l) [wave][16 MB]; then the ancestor masks if they are held here
    extern __shared__ __attribute__((aligned(16))) float merge_lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const int kg = DR_WAVES / rg;
    const int rgi = wave % rg, kgi = wave / rg;
    const int work = xcd_work_index(p.B * p.Hkv * p.n_splits * p.n_row_tiles);
    if (work < 0) return;                                         // grid padding (whole workgroup)
    const int rt = work % p.n_row_tiles, unit = work / p.n_row_tiles;
    const int split = unit % p.n_splits;
    const int g = (unit / p.n_splits) % p.Hkv, b = unit / (p.n_splits * p.Hkv);

    const int n_raw = p.n_nodes[b];
    const int P_raw = p.prefix_len[b];
    const int r_base = (rt * rg + rgi) * (16 * MB);
    typename Ops::Q q[MB];
    uintx4 mw[MB];                              // ancestor mask of the row's node
    int node[MB];
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
        const int r = r_base + rb * 16 + l16;
        const int rc = r < p.R ? r : 0;
        node[rb] = (rc * p.g_magic) >> 16;
        const int hl = rc - node[rb] * p.G;
        Ops::load_q(q[rb], static_cast<const T*>(p.q) +
                    ((static_cast<size_t>(b) * p.K_max + node[rb]) * p.Hq + (g * p.G + hl)) * D, lg);
        if constexpr (MASK_HELD)
            mw[rb] = *reinterpret_cast<const uintx4*>(p.mask + (static_cast<size_t>(b) * p.K_max + node[rb]) * GRAFT_MASK_WORDS);
    }

    uintx4* mask_lds = reinterpret_cast<uintx4*>(merge_lds + (kg == 1 ? 0 : DR_WAVES * 16 * MB * (PITCH + 2)));
    if constexpr (!MASK_HELD) {
        static_assert(GRAFT_MAX_NODES * 4 <= DR_THREADS, "one mask word per thread");
        if (tid < p.K_max * 4)
            reinterpret_cast<unsigned*>(mask_lds)[tid] =
                reinterpret_cast<const unsigned*>(p.mask + static_cast<size_t>(b) * p.K_max * GRAFT_MASK_WORDS)[tid];
        __syncthreads();
    }

    int n = n_raw;
    if (n < 1 || n > p.K_max) n = 0;
    const int cap = p.max_pages * GRAFT_PAGE_SIZE;
    int P = P_raw;
    P = P < 0 ? 0 : (P > cap ? cap : P);
    const int total = n ? ((P + n) < cap ? (P + n) : cap) : 0;
    const int n_tiles = (total + TK - 1) / TK;
    const int per_split = (n_tiles + p.n_splits - 1) / p.n_splits;
    const int tile0 = split * per_split;
    const int tile1 = (tile0 + per_split) < n_tiles ? (tile0 + per_split) : n_tiles;
    // this wavefront's tiles: tile0 + kgi, + kg, ...; none if all its rows belong to absent nodes
    const int first = tile0 + kgi;
    const bool rows_live = ((r_base * p.g_magic) >> 16) < n && r_base < p.R;
    const int count = (rows_live && first < tile1) ? (tile1 - first + kg - 1) / kg : 0;

    float m[MB], l[MB];
    floatx4 lv[MB];                             // row sums where the matrix cores take them (every entry the row's sum)
    floatx4 o[MB][NO];
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
        m[rb] = -INFINITY;
        l[rb] = 0.f;
        lv[rb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < NO; ++e) o[rb][e] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

    if (count > 0) {
        constexpr int PAGES = TK / GRAFT_PAGE_SIZE, TPR = 64 / PAGES;      // pages per tile, tiles per table register
        const int last = total - 1, last_pg = last >> 4;
        const int32_t* table = p.block_table + static_cast<size_t>(b) * p.max_pages;
        const char* kc = static_cast<const char*>(p.k) + static_cast<int64_t>(g) * p.head_stride * sizeof(T);
        const char* vc = static_cast<const char*>(p.v) + static_cast<int64_t>(g) * p.head_stride * sizeof(T);
        const unsigned ts = static_cast<unsigned>(p.token_stride) * sizeof(T);   // bytes
        int tb = 0;
        // Tiles in the order they are taken: the wavefront's last one first, so that the one tile of
        // the sequence that can reach past its end is only ever the first of a wavefront.  Loads
        // inside the loop then need no branch; with one, the compiler no longer knows how many
        // transfers are in flight and waits for most of what it has just requested.
        auto tile_at = [&](int it) { return first + kg * (it == 0 ? count - 1 : it - 1); };
        auto load_table = [&](int it) {
            const int pg = tile_at(it + lane / PAGES) * PAGES + lane % PAGES;
            tb = table[pg < last_pg ? pg : last_pg];
        };
        // (the wavefront-uniform part of an address is scalar, the lane's part loop-invariant)
        auto page_base = [&](int it, int c) {
            return static_cast<int64_t>(__builtin_amdgcn_readlane(tb, (it & (TPR - 1)) * PAGES + c)) * p.page_stride * static_cast<int64_t>(sizeof(T));
        };
        const unsigned k_off = l16 * ts + Ops::k_lane(lg), v_off = 4 * lg * ts + Ops::v_lane(l16);
        auto load_keys = [&](typename Ops::K& t, int it) {
#pragma unroll
            for (int c = 0; c < NC; ++c) Ops::load_k(t, c, kc + page_base(it, c), k_off);
        };
        auto load_values = [&](typename Ops::V& t, int it) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    Ops::load_v(t, c, i, vc + page_base(it, c) + static_cast<int64_t>(i) * ts, v_off);
        };
        // a tile that may reach past the end: keys past the last token read the last token again
        // (its values are finite, and its probability there is zero)
        auto load_clamped = [&](typename Ops::K& kt, typename Ops::V& vt, int it) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int t_page = tile_at(it) * TK + 16 * c;
                const int lim = last - (t_page < last ? t_page : (last & ~15));
                Ops::load_k(kt, c, kc + page_base(it, c), static_cast<unsigned>(l16 < lim ? l16 : lim) * ts + Ops::k_lane(lg));
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int k = 4 * lg + i;
                    Ops::load_v(vt, c, i, vc + page_base(it, c), static_cast<unsigned>(k < lim ? k : lim) * ts + Ops::v_lane(l16));
                }
            }
        };
        const float sc = p.scale_log2e;
        // One tile, in kt and vt.  With one register set (!DOUBLE) the next tile's keys and values are
        // requested here, each as soon as the current ones are out of their registers.
        auto step = [&](typename Ops::K& kt, typename Ops::V& vt, int it, auto more_) {
            constexpr bool more = decltype(more_)::value && !DOUBLE;
            const int t0 = tile_at(it) * TK;
            const bool masked = t0 + TK > P;
            floatx4 s[MB][NC];
#pragma unroll
            for (int rb = 0; rb < MB; ++rb) Ops::scores(kt, q[rb], s[rb]);
            if constexpr (more) load_keys(kt, it + 1);
            if (__builtin_expect(masked, 0)) {
#pragma unroll
                for (int rb = 0; rb < MB; ++rb) {
                    if constexpr (!MASK_HELD) mw[rb] = mask_lds[node[rb]];
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int j = t0 + 16 * c + 4 * lg + i - P;            // tree slot
                            const int wi = (j >> 5) & 3;
                            const unsigned word = wi == 0 ? mw[rb][0] : (wi == 1 ? mw[rb][1] : (wi == 2 ? mw[rb][2] : mw[rb][3]));
                            const bool valid = (j < 0) | ((j < n) & ((word >> (j & 31)) & 1u));
                            s[rb][c][i] = valid ? s[rb][c][i] : -INFINITY;
                        }
                }
            }
            float mx[MB];
            bool raise = false;
#pragma unroll
            for (int rb = 0; rb < MB; ++rb) {
                float x = fmaxf(fmaxf(s[rb][0][0], s[rb][0][1]), fmaxf(s[rb][0][2], s[rb][0][3]));
                if constexpr (NC == 2)
                    x = fmaxf(x, fmaxf(fmaxf(s[rb][1][0], s[rb][1][1]), fmaxf(s[rb][1][2], s[rb][1][3])));
                mx[rb] = x * sc;
                raise = raise || mx[rb] > m[rb] + DR_LAZY_LOG2;
            }
            // (rare) a row without a reference, or one that outgrew it: raise it to the maximum seen
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {
#pragma unroll
                for (int rb = 0; rb < MB; ++rb) {
                    const float mn = fmaxf(m[rb], rows_max_f32(mx[rb]));
                    const float a = mn == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m[rb] - mn);
                    m[rb] = mn;
                    l[rb] *= a;
                    if constexpr (Ops::SUM_MFMA) lv[rb] *= a;
#pragma unroll
                    for (int e = 0; e < NO; ++e) o[rb][e] *= a;
                }
            }
            typename Ops::A va;
            Ops::arrange(vt, va);
            if constexpr (more && Ops::FREES_V) load_values(vt, it + 1);
#pragma unroll
            for (int rb = 0; rb < MB; ++rb) {
                const float neg = m[rb] == -INFINITY ? 0.f : -m[rb];
                float sum = 0.f;
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        s[rb][c][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[rb][c][i], sc, neg));
                        if constexpr (!Ops::SUM_MFMA) sum += s[rb][c][i];
                    }
                l[rb] += sum;
                Ops::accumulate(vt, va, s[rb], o[rb], lv[rb]);
            }
            if constexpr (more && !Ops::FREES_V) load_values(vt, it + 1);
        };
        // chunks of the tiles that one table register covers
        for (int it = 0; it < count;) {
            const int end = it + TPR < count ? it + TPR : count;
            typename Ops::K ka, kb;
            typename Ops::V va, vb;
            load_table(it);
            load_clamped(ka, va, it);
            if constexpr (DOUBLE) {
                for (; it + 2 < end; it += 2) {
                    load_keys(kb, it + 1);
                    load_values(vb, it + 1);
                    step(ka, va, it, std::false_type{});
                    load_keys(ka, it + 2);
                    load_values(va, it + 2);
                    step(kb, vb, it + 1, std::false_type{});
                }
                if (it + 1 < end) {
                    load_keys(kb, it + 1);
                    load_values(vb, it + 1);
                    step(ka, va, it, std::false_type{});
                    step(kb, vb, it + 1, std::false_type{});
                } else {
                    step(ka, va, it, std::false_type{});
                }
            } else {
                for (; it + 1 < end; ++it) step(ka, va, it, std::true_type{});
                step(ka, va, it, std::false_type{});
            }
            it = end;
        }
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) l[rb] = Ops::SUM_MFMA ? lv[rb][0] : rows_sum_f32(l[rb]);
    }

    // ---- results: this workgroup's rows, merged over its key groups
    T* outp = static_cast<T*>(p.out);
    float* ws_o = reinterpret_cast<float*>(p.ws_o);
    const size_t part = ((static_cast<size_t>(b) * p.Hkv + g) * p.n_splits + split) * p.R_pad;
    if (kg == 1) {
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) {
            const int r = r_base + rb * 16 + l16;
            if (p.n_splits == 1) {
                const bool keep = r < p.R && node[rb] < n && l[rb] > 0.f;
                const float inv = keep ? 1.0f / l[rb] : 0.f;
                T* row = outp + ((static_cast<size_t>(b) * p.K_max + node[rb]) * p.Hq + g * p.G + (r - node[rb] * p.G)) * D;
                if (r < p.R) {
#pragma unroll
                    for (int u = 0; u < D / 16; ++u) {
                        floatx4 x = Ops::piece(o[rb], u) * inv;
                        if (!keep) x = floatx4{0.f, 0.f, 0.f, 0.f};
                        store4(row + Ops::dim(u, lg), x);
                    }
                }
            } else {
#pragma unroll
                for (int u = 0; u < D / 16; ++u) store4(ws_o + (part + r) * D + Ops::dim(u, lg), Ops::piece(o[rb], u));
                if (lg == 0) {
                    p.ws_ml[2 * (part + r)] = m[rb];
                    p.ws_ml[2 * (part + r) + 1] = l[rb];
                }
            }
        }
        return;
    }
    float* ml_lds = merge_lds + DR_WAVES * 16 * MB * PITCH;
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
        float* row = merge_lds + ((wave * MB + rb) * 16 + l16) * PITCH;
#pragma unroll
        for (int u = 0; u < D / 16; ++u) store4(row + Ops::dim(u, lg), Ops::piece(o[rb], u));
        if (lg == 0) {
            ml_lds[2 * ((wave * MB + rb) * 16 + l16)] = m[rb];
            ml_lds[2 * ((wave * MB + rb) * 16 + l16) + 1] = l[rb];
        }
    }
    __syncthreads();
    const int rows = rg * 16 * MB;                                // of this workgroup
    for (int x = tid; x < rows * (D / 4); x += DR_THREADS) {
        const int lr = x / (D / 4), d4 = x % (D / 4);
        float mm = -INFINITY;
        for (int k = 0; k < kg; ++k) mm = fmaxf(mm, ml_lds[2 * (k * rows + lr)]);
        float den = 0.f;
        floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int k = 0; k < kg; ++k) {
            const float mk = ml_lds[2 * (k * rows + lr)];
            const float f = mk == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mk - mm);
            den += f * ml_lds[2 * (k * rows + lr) + 1];
            acc += *reinterpret_cast<const floatx4*>(merge_lds + (k * rows + lr) * PITCH + 4 * d4) * f;
        }
        const int r = rt * rows + lr;
        if (p.n_splits == 1) {
            if (r < p.R) {
                const int i = (r * p.g_magic) >> 16;
                const bool keep = i < n && den > 0.f;
                const floatx4 y = keep ? acc * (1.0f / den) : floatx4{0.f, 0.f, 0.f, 0.f};
                store4(outp + ((static_cast<size_t>(b) * p.K_max + i) * p.Hq + g * p.G + (r - i * p.G)) * D + 4 * d4, y);
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

// Merge of the splits: one thread per four dims of a row, the splits' pieces requested eight at a time.
template <typename T, int D>
__global__ __launch_bounds__(256) void tree_attn_direct_merge_kernel(AttnParams p, int32_t n_rows) {
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int row = x / (D / 4), d4 = x % (D / 4);                // row over B * Hkv * R
    if (row >= n_rows) return;
    const int r = row % p.R, bg = row / p.R, g = bg % p.Hkv, b = bg / p.Hkv;
    const int n_raw = p.n_nodes[b];
    const size_t base = static_cast<size_t>(bg) * p.n_splits * p.R_pad + r;
    const float* ws_o = reinterpret_cast<const float*>(p.ws_o);
    float mm = -INFINITY, den = 0.f;
    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < p.n_splits; s0 += 8) {
        floatx4 ov[8];
        float mv[8], lv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            ov[u] = floatx4{0.f, 0.f, 0.f, 0.f};
            mv[u] = -INFINITY;
            lv[u] = 0.f;
            if (s0 + u < p.n_splits) {
                const size_t i = base + static_cast<size_t>(s0 + u) * p.R_pad;
                mv[u] = p.ws_ml[2 * i];
                lv[u] = p.ws_ml[2 * i + 1];
                ov[u] = *reinterpret_cast<const floatx4*>(ws_o + i * D + 4 * d4);
            }
        }
        float mx = mm;
#pragma unroll
        for (int u = 0; u < 8; ++u) mx = fmaxf(mx, mv[u]);
        if (mx == -INFINITY) continue;
        const float keep = mm == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mm - mx);
        den *= keep;
        acc *= keep;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float f = mv[u] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mv[u] - mx);
            den += f * lv[u];
            acc += ov[u] * f;
        }
        mm = mx;
    }
    int n = n_raw;
    if (n < 1 || n > p.K_max) n = 0;
    const int i = (r * p.g_magic) >> 16;
    const bool keep = i < n && den > 0.f;
    const floatx4 y = keep ? acc * (1.0f / den) : floatx4{0.f, 0.f, 0.f, 0.f};
    store4(static_cast<T*>(p.out) + ((static_cast<size_t>(b) * p.K_max + i) * p.Hq + g * p.G + (r - i * p.G)) * D + 4 * d4, y);
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
static size_t direct_lds_bytes(int mb, int rg, int D) {
    const size_t merge = rg == DR_WAVES ? 0 : static_cast<size_t>(DR_WAVES) * 16 * mb * (D + 4 + 2) * sizeof(float);
    return merge + (mb > 2 ? GRAFT_MAX_NODES * GRAFT_MASK_WORDS * sizeof(u64) : 0);
}

// Launch shape: row blocks per wavefront, row groups per workgroup and splits that make the
// estimated time smallest.  One workgroup of eight wavefronts (two per SIMD) is resident per
// compute unit, so the job runs in ceil(workgroups / CUs) rounds of a fixed part plus the tiles of
// a wavefront, times two for the SIMD's other wavefront.
DirectPlan plan_direct(int32_t B, int32_t K_max, int32_t Hq, int32_t Hkv, int32_t D, int32_t max_pages, int32_t dtype,
                       bool may_split) {
    DirectPlan best{};
    best.cost = -1.0;
    const int R = K_max * (Hq / Hkv), blocks = (R + 15) / 16;
    const int TK = dtype == GRAFT_F32 ? 16 : 32;
    const int64_t tiles = (static_cast<int64_t>(max_pages) * GRAFT_PAGE_SIZE + TK - 1) / TK;
    const int64_t cus = device_compute_units();
    const int mb_max = dtype == GRAFT_F32 ? (D == 128 ? 1 : 2) : 4;   // (what the registers hold)
    for (int mb = 1; mb <= mb_max; mb *= 2) {
        const double c_tile = 2.0 * (dtype == GRAFT_F32 ? 200.0 + mb * D * 16.5 : 150.0 + mb * 350.0);
        for (int rg = 1; rg <= DR_WAVES; rg *= 2) {
            const int kg = DR_WAVES / rg;
            const int n_rt = (blocks + rg * mb - 1) / (rg * mb);
            if (rg > 1 && (rg / 2) * mb >= blocks) break;          // half the row groups would do
            const int64_t units = static_cast<int64_t>(B) * Hkv * n_rt;
            for (int sp = 1; sp <= (may_split ? DR_MAX_SPLITS : 1); ++sp) {
                const int64_t per = (tiles + static_cast<int64_t>(sp) * kg - 1) / (static_cast<int64_t>(sp) * kg);
                const int64_t rounds = (units * sp + cus - 1) / cus;
                const double rows = static_cast<double>(B) * Hkv * R;
                const double cost = rounds * (9000.0 + per * c_tile) + (sp > 1 ? 8000.0 + sp * rows * D / (256.0 * 10.0) : 0.0);
                if (best.cost < 0.0 || cost < best.cost) {
                    best.cost = cost;
                    best.mb = mb;
                    best.rg = rg;
                    best.n_row_tiles = n_rt;
                    best.n_splits = sp;
                }
                if (units * sp > 4 * cus || per <= 1) break;
            }
        }
    }
    best.r_pad = best.n_row_tiles * best.rg * best.mb * 16;
    if (best.n_splits > 1) {
        const size_t rows = static_cast<size_t>(B) * Hkv * best.n_splits * best.r_pad;
        best.ws_o_bytes = rows * D * sizeof(float);
        best.ws_bytes = best.ws_o_bytes + rows * 2 * sizeof(float);
    }
    return best;
}

template <typename T, int D, int MB>
static int32_t launch_one(const DirectPlan& pl, const AttnParams& p, hipStream_t s) {
    auto kernel = tree_attn_direct_kernel<T, D, MB>;
    const unsigned lds = static_cast<unsigned>(direct_lds_bytes(MB, pl.rg, D));
    if (lds > 65536) {                                            // more than the default limit needs opting in, once per device
        static thread_local int done_device = -1;
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) dev = 0;
        if (done_device != dev) {
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            done_device = dev;
        }
    }
    const dim3 grid(xcd_grid(static_cast<int64_t>(p.B) * p.Hkv * pl.n_splits * pl.n_row_tiles));
    launch_main(kernel, grid, dim3(DR_THREADS), lds, s, p, pl.rg);
    int32_t rc = check_launch();
    if (rc != GRAFT_OK || pl.n_splits == 1) return rc;
    const int64_t n_rows = static_cast<int64_t>(p.B) * p.Hkv * p.R;
    if (n_rows * (D / 4) > 0x7fffffff) return GRAFT_ERR_SHAPE;
    hipLaunchKernelGGL((tree_attn_direct_merge_kernel<T, D>), dim3(static_cast<unsigned>((n_rows * (D / 4) + 255) / 256)), dim3(256), 0, s,
                       p, static_cast<int32_t>(n_rows));
    return check_launch();
}

int32_t launch_direct(const DirectPlan& pl, AttnParams p, int32_t D, int32_t dtype, void* workspace, hipStream_t s) {
    p.n_splits = pl.n_splits;
    p.n_row_tiles = pl.n_row_tiles;
    p.R_pad = pl.r_pad;
    p.ws_o = static_cast<unsigned short*>(workspace);
    p.ws_ml = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + pl.ws_o_bytes);
    if (dtype == GRAFT_F32) {
        if (D == 64) return pl.mb == 1 ? launch_one<float, 64, 1>(pl, p, s) : launch_one<float, 64, 2>(pl, p, s);
        return launch_one<float, 128, 1>(pl, p, s);
    }
    if (pl.mb == 4) return launch_one<__bf16, 64, 4>(pl, p, s);
    return pl.mb == 1 ? launch_one<__bf16, 64, 1>(pl, p, s) : launch_one<__bf16, 64, 2>(pl, p, s);
}

}  // namespace graft
