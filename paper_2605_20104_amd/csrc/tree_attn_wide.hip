// graft_tree_attn, MFMA path with row blocks of 32 (bf16, D = 128): tiles of 192, 256 and 384 rows, and of 128 as a kernel of its own
// (tree_attn_wide_128.hip, which compiles this file once more).
//
// The same split-KV scheme as tree_attn_mfma_kernel (tree_attn.hip: 256 threads, one workgroup per compute unit, 64-token
// stages from memory straight to an LDS ring of four, partial rows for the merge kernel), with another loop.
//   why   : the 16-row kernel is bound by issue slots: beside a 16x16x32 MFMA one exp2 or two plain instructions are free, beside a
//           32x32x16, twice the products, three or six.  And it reads every K and V operand from LDS once per wavefront,
//           for the wavefront's 48 rows where a tile has 192; here an operand serves 96.
//   tiles : a wavefront has NB blocks of 32 rows.  KEYS: two wavefronts share their blocks and take every other 32-token
//           sub-tile (2 NB blocks a tile); what they add up is merged through LDS behind the loop.  ROWS: every wavefront has its
//           own blocks and takes all sub-tiles (4 NB blocks).  384 rows halve the transfers of two tiles of 192 and double the
//           partial rows, which pays for long splits.
//   loop  : a unit is (sub-tile, row block).  In phase u the matrix cores multiply S^T = K Q^T of unit u and O^T += V^T P^T of unit
//           u - 2 in turn, 8 MFMAs each, while the vector ALUs turn the scores of unit u - 1 into probabilities; a slot holds one
//           MFMA, one fma, one exp2, one addition and half a pack.  The K and V operands of a sub-tile stay in
//           registers for its NB units and are replaced one by one behind their last use, a phase ahead of their first.
//           Lane (half, l32) of a score tile has row l32 and 16 of the tokens, which are already laid out as the B operand of the
//           second product (tokens 8 (v / 4) + 4 half + v % 4); its A operand comes from the LDS transpose read in that order.
//   stages: one barrier a stage.  The transfers of stage k + 3 go between the MFMAs (a third of the slots of 24; in one burst
//           behind the barrier they cost 560 cycles of 2900 a stage), through buffer descriptors that end with the page's
//           last token, so that whole, last and absent pages are the same eight instructions.  The loop over stages that lie
//           inside the prefix has no branch but its own; the first stage and those with tree slots have copies of their own.
//   sums  : of the probabilities as they leave exp2, in fp32: rounded ones would need an unpacking each or the matrix
//           cores (v_dot2 holds those too, 18 cycles an instruction).  Queries are not scaled and rounded again: the softmax
//           scale is applied to the scores in fp32.  Together that is closer to a 64-bit reference than the 16-row kernel.
//   range : a row's reference is fixed by the first sub-tile of which it sees anything: zero where the maximum lies in 0 .. 16 (log2
//           units), else that maximum, so that its sum is never below about one.  Behind every stage rows whose sum has passed
//           2^24 move theirs up by a power of two (exact).  Sums and products that left the range of fp32 in between are seen
//           there; what the last two units of a split add is seen behind the loop, where sums from 2^26 on do not pass: below, products
//           with values of up to 2^100 are finite.  A wavefront with such a row, or with one that sees tokens and has no
//           sum, makes the workgroup go over its keys once more, that wavefront with the exact running maximum.
//
// Measured (MI355X, N(0,1) operands, all compute units busy).  Cycles of a stage of 192 rows 3160 -> 2220, of which 1540 are
// MFMAs.  The chip lowers its clock with the load (2.38 -> 1.9 GHz on 33 stages, 1.85 -> 1.55 on 257), so the time follows the
// energy as much as the cycles.  us a call, 16-row kernel -> this one: 8 sequences of 4096 keys, 48 x 64 heads on 4: 56.6 -> 53.3
// (1024 keys: 25.2 -> 24.0); 4 of 65536, 96 x 32 heads on 8: 408 -> 365 (384 rows); one of 16384: 35.7 -> 33.4; 8 of 16000, 64 x 32
// heads on 8 (256 rows): 137.1 -> 133.2; 4 of 20440, 40 x 32 heads on 4 (three tiles of 128 rows): 82.7 -> 67.0.  Tried and dropped: 320 rows as two blocks a wavefront and a third for every other
// sub-tile (62 against 77 thousand cycles for 17 stages, and 65.4 against 63.9 us a round with 32K keys: the clock);
// row sums through v_dot2_f32_bf16 or 4x4x4 MFMAs (678 and 596 cycles a phase, 530 with additions).
#include "attn_mfma.h"

// (the body in a function of its own, called by both kernels, cost the others 2.5 per cent: other registers)
#ifdef GRAFT_WIDE_128
#define GRAFT_WIDE_KERNEL tree_attn_wide_128_kernel
#else
#define GRAFT_WIDE_KERNEL tree_attn_wide_kernel
#endif

namespace graft {

enum WideMode { WIDE_ROWS = 1, WIDE_KEYS = 2 };
constexpr int WD_BLOCK = 32;                    // query rows of a row block
constexpr float WD_LAZY_SUM = 16777216.0f;      // a row keeps its reference while its sum stays below 2^24
constexpr float WD_SMALL_SCORE = 16.0f;         // rows whose first scores stay below this (log2 units), and reach zero, need no reference
constexpr float WD_MIN_SUM = 0.5f, WD_MAX_SUM = 67108864.0f;    // sums that need no second pass (2^26; regular ones end below 2 x 2^24)

template <int NB_, int MODE_> struct WideShape {
    static constexpr int NB = NB_, MODE = MODE_;
    static constexpr int UNITS = MODE == WIDE_ROWS ? 2 * NB : NB;                 // of a wavefront in a stage
    static constexpr int TILE_ROWS = (MODE == WIDE_ROWS ? 4 : 2) * NB * WD_BLOCK;
    static constexpr int wrap(int u) { return (u + 2 * UNITS) % UNITS; }
    static constexpr int block(int u) { return u % NB; }
    static constexpr int visit(int u) { return u / NB; }          // first or second sub-tile of the stage that the wavefront takes
    static constexpr bool last_of_sub(int u) { return block(u) == NB - 1; }
    static constexpr bool SHARED = MODE == WIDE_KEYS;
    static __device__ __forceinline__ int sub_tile(int v, int kg) { return SHARED ? kg : v; }
    static __device__ __forceinline__ int row0(int b, int wave) { return ((SHARED ? wave >> 1 : wave) * NB + b) * WD_BLOCK; }
};

// AccVGPRs: O^T of row block b, dims 32 e ..: a[64 b + 16 e ..]; Q' of row blocks 0 and 1, dim step d: a[64 NB + 32 b + 4 d ..]
constexpr int wide_o(int b, int e) { return 64 * b + 16 * e; }
template <int NB> constexpr int wide_q(int b, int d) { return 64 * NB + 32 * b + 4 * d; }
template <int NB> constexpr int wide_acc_used() { return 64 * NB + 64; }

template <int NB> __device__ __forceinline__ void reserve_wide_registers() {
    asm volatile("" ::: GRAFT_ACC_BLOCK_0);
    asm volatile("" ::: GRAFT_ACC_BLOCK_1);
    asm volatile("" ::: GRAFT_ACC_BLOCK_2);
    asm volatile("" ::: GRAFT_ACC_BLOCK_3);
    if constexpr (wide_acc_used<NB>() > 192) {
        asm volatile("" ::: GRAFT_ACC_BLOCK_4);
        asm volatile("" ::: GRAFT_ACC_BLOCK_5);
    }
}

template <int NB> struct WideState {
    floatx16 s[NB];
    uintx4 p[NB][2];
    bf16x8 k[8], v[8];
    bf16x8 q2[NB == 3 ? 8 : 1];
    float l[NB], negm[NB];
};

template <int QR, bool FIRST, bool GUARD>
__device__ __forceinline__ void mfma_s_acc(floatx16& d, const bf16x8& k) {
    if constexpr (FIRST && GUARD) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], 0" : "=&v"(d) : "v"(k), "n"(QR), "n"(QR + 3));
    else if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], 0" : "=&v"(d) : "v"(k), "n"(QR), "n"(QR + 3));
    else if constexpr (GUARD) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], %0" : "+v"(d) : "v"(k), "n"(QR), "n"(QR + 3));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], %0" : "+v"(d) : "v"(k), "n"(QR), "n"(QR + 3));
}
template <bool FIRST, bool GUARD>
__device__ __forceinline__ void mfma_s_vgpr(floatx16& d, const bf16x8& k, const bf16x8& q) {
    if constexpr (FIRST && GUARD) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(k), "v"(q));
    else if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(k), "v"(q));
    else if constexpr (GUARD) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(k), "v"(q));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(k), "v"(q));
}
template <int NB, int B, int D, bool GUARD> __device__ __forceinline__ void mfma_s(WideState<NB>& w, const bf16x8& k) {
    if constexpr (B < 2) mfma_s_acc<wide_q<NB>(B, D), D == 0, GUARD>(w.s[B], k);
    else mfma_s_vgpr<D == 0, GUARD>(w.s[B], k, w.q2[D]);
}
template <int OR, bool GUARD> __device__ __forceinline__ void mfma_wide_o(const bf16x8& v, const uintx4& p) {
    if constexpr (GUARD) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 a[%0:%1], %2, %3, a[%0:%1]" : : "n"(OR), "n"(OR + 15), "v"(v), "v"(p));
    else asm volatile("v_mfma_f32_32x32x16_bf16 a[%0:%1], %2, %3, a[%0:%1]" : : "n"(OR), "n"(OR + 15), "v"(v), "v"(p));
}

__device__ __forceinline__ bf16x8 read_k(unsigned base, int d) {
    return *reinterpret_cast<const bf16x8 __attribute__((address_space(3)))*>(static_cast<size_t>(base ^ (static_cast<unsigned>(d) << 5)));
}
// operand n = 4 kk + e
__device__ __forceinline__ bf16x8 read_v(unsigned base, int n) {
    bf16x8 v;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const short4_t r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (short4_t __attribute__((address_space(3)))*)(static_cast<size_t>((base ^ (static_cast<unsigned>(n & 3) << 6)) +
                                                                              (16 * (n >> 2) + 8 * c) * AT_ROW_BYTES)));
        const bf16x4 r4 = __builtin_bit_cast(bf16x4, r);
        v[4 * c] = r4[0];
        v[4 * c + 1] = r4[1];
        v[4 * c + 2] = r4[2];
        v[4 * c + 3] = r4[3];
    }
    return v;
}
// sum and maximum over the two lanes that hold the same row
__device__ __forceinline__ float pair_sum(float v) {
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float pair_max(float v) {
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The lane index for rare paths: what is computed from it stays there instead of in registers across the loop.
__device__ __forceinline__ int opaque_lane() {
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return lane;
}

// A value that is computed where it is written in the source: the compiler would move it to where it is used, behind the phase.
template <class T> __device__ __forceinline__ T pinned(T x) {
    asm volatile("" : "+v"(x));
    return x;
}

// One phase: scores of unit J, probabilities of unit J - 1, products of unit J - 2.  extra(slot) adds to a slot.  530 cycles where the
// MFMAs alone take 514, with the LDS reads 550.
template <class S, int J, bool QK, bool SM, bool PV, class Extra>
__device__ __forceinline__ void phase(WideState<S::NB>& w, float c_log2, unsigned k_next, unsigned v_next, Extra&& extra) {
    constexpr int NB = S::NB, QB = S::block(S::wrap(J)), SB = S::block(S::wrap(J - 1)), PB = S::block(S::wrap(J - 2));
    constexpr bool K_RELOAD = QK && S::last_of_sub(S::wrap(J)), V_RELOAD = QK && S::last_of_sub(S::wrap(J - 2));      // (for the next sub-tile)
    float e[16];
    static_for<0, 16>([&](auto i_) {
        GRAFT_CONST(i, i_);
        constexpr int h = i >> 1;
        if constexpr (i % 2 == 0) {
            if constexpr (QK) mfma_s<NB, QB, h, i == 0>(w, w.k[h]);
        } else {
            if constexpr (PV) mfma_wide_o<wide_o(PB, h & 3), i == 1>(w.v[h], w.p[PB][h >> 2]);
        }
        if constexpr (SM) {
            if constexpr (i == 1) e[0] = pinned(__builtin_amdgcn_exp2f(__builtin_fmaf(w.s[SB][0], c_log2, w.negm[SB])));
            if constexpr (i >= 1) e[i] = pinned(__builtin_amdgcn_exp2f(__builtin_fmaf(w.s[SB][i], c_log2, w.negm[SB])));
            if constexpr (i == 2) w.l[SB] = pinned(w.l[SB] + e[0]);
            if constexpr (i >= 2) w.l[SB] = pinned(w.l[SB] + e[i - 1]);
            if constexpr (i >= 2 && i % 2 == 0) w.p[SB][(h - 1) >> 2][(h - 1) & 3] = pinned(pack_bf16(e[i - 2], e[i - 1]));
        }
        if constexpr (K_RELOAD && i % 2 == 1) w.k[h] = read_k(k_next, h);
        if constexpr (V_RELOAD && i % 2 == 0 && i >= 2) w.v[h - 1] = read_v(v_next, h - 1);
        extra(i_);
        __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (SM) {
        w.p[SB][1][3] = pinned(pack_bf16(e[14], e[15]));
        w.l[SB] = pinned(w.l[SB] + e[15]);
    }
    if constexpr (V_RELOAD) w.v[7] = read_v(v_next, 7);
    __builtin_amdgcn_sched_barrier(0);
}

// Scores that reach past the prefix: what the row does not see becomes -inf.
__device__ __forceinline__ unsigned row_window(int r, int t_sub, int P, int n, int slots, int R, int g_magic, const unsigned* Ms) {
    const int node = (r * g_magic) >> 16;
    const unsigned* row = Ms + 4 * (r < R && node < n ? node : 0);
    return visible_window(t_sub - P, slots, [&](int k) { return row[k]; });
}
__device__ __forceinline__ void mask_scores(floatx16& s, unsigned win, int half) {
    win >>= 4 * half;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = keep_visible(s[v], win, 8 * (v >> 2) + (v & 3));
}
__device__ __forceinline__ float score_max(const floatx16& s) {
    float mx = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = __builtin_fmaxf(mx, s[v]);
    return pair_max(mx);
}
__device__ __forceinline__ void settle(floatx16& s) { asm volatile("s_nop 15\n\ts_nop 7" : "+v"(s)); }

// Rows whose sums have grown: reference up by a power of two, everything accumulated down by it (exact).  PEND: the row block
// whose probabilities are not multiplied yet.
template <class S>
__device__ __forceinline__ bool raise_rows(WideState<S::NB>& w) {
    constexpr int PEND = S::block(S::wrap(S::UNITS - 2));
    GRAFT_MFMA_SETTLE();
    float odd = 0.f;
    static_for<0, S::NB>([&](auto b_) {
        GRAFT_CONST(b, b_);
        const float lt = pair_sum(w.l[b]);
        const int ex = static_cast<int>((__float_as_uint(lt) >> 23) & 0xffu) - 127;
        const int shift = ex >= 23 && ex < 128 ? ex : 0;
        const float f = __uint_as_float(static_cast<unsigned>(127 - shift < 1 ? 1 : 127 - shift) << 23);
        odd = __builtin_fmaf(lt, 0.f, odd);
        w.negm[b] -= static_cast<float>(shift < 126 ? shift : 126);
        w.l[b] *= f;
        if constexpr (b == PEND) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int j = 0; j < 4; ++j) w.p[b][kk][j] = scale_bf16_pair(w.p[b][kk][j], f);
        }
        static_for<0, 64>([&](auto k_) {
            GRAFT_CONST(k, k_);
            const float o = acc_get<wide_o(b, 0) + k>() * f;
            odd = __builtin_fmaf(o, 0.f, odd);
            acc_set<wide_o(b, 0) + k>(o);
        });
    });
    GRAFT_MFMA_SETTLE();
    return __builtin_amdgcn_ballot_w64(!(odd == 0.f)) != 0;
}

// Exact running maximum, one unit at a time.
template <class S, int B>
__device__ __forceinline__ void exact_unit(WideState<S::NB>& w, unsigned k_addr, unsigned v_addr, bool masked, unsigned win, int half, float c_log2) {
    constexpr int NB = S::NB;
    static_for<0, 8>([&](auto d_) {
        GRAFT_CONST(d, d_);
        w.k[d] = read_k(k_addr, d);
        w.v[d] = read_v(v_addr, d);
    });
    asm volatile("s_nop 7" ::: "memory");
    static_for<0, 8>([&](auto d_) {
        GRAFT_CONST(d, d_);
        mfma_s<NB, B, d, true>(w, w.k[d]);
        asm volatile("s_nop 15" ::: "memory");
    });
    settle(w.s[B]);
    if (masked) mask_scores(w.s[B], win, half);
    const float m = -w.negm[B], mn = __builtin_fmaxf(m, score_max(w.s[B]) * c_log2);
    const float a = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mn);
    const float neg = mn == -INFINITY ? 0.f : -mn;
    w.negm[B] = -mn;
    w.l[B] *= a;
    static_for<0, 64>([&](auto k_) {
        GRAFT_CONST(k, k_);
        acc_scale<wide_o(B, 0) + k>(a);
    });
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(w.s[B][2 * j], c_log2, neg)), e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(w.s[B][2 * j + 1], c_log2, neg));
        w.p[B][j >> 2][j & 3] = pack_bf16(e0, e1);
        w.l[B] += e0 + e1;
    }
    GRAFT_MFMA_SETTLE();
    static_for<0, 8>([&](auto n_) {
        GRAFT_CONST(n, n_);
        mfma_wide_o<wide_o(B, n & 3), true>(w.v[n], w.p[B][n >> 2]);
        asm volatile("s_nop 15" ::: "memory");
    });
    GRAFT_MFMA_SETTLE();
    GRAFT_KEEP(w.p[B][0]);
    GRAFT_KEEP(w.p[B][1]);
}

template <int NB, int MODE>
__global__ __launch_bounds__(AT_THREADS) void GRAFT_WIDE_KERNEL(GRAFT_ATTN_ARGS) {
    using S = WideShape<NB, MODE>;
    constexpr int UNITS = S::UNITS;
    __shared__ __attribute__((aligned(1024))) unsigned char kv[AT_NBUF][AT_STAGE_BYTES];
    __shared__ unsigned Ms[GRAFT_MAX_NODES * GRAFT_MASK_WORDS * 2];   // ancestor masks as 32-bit words
    __shared__ int32_t Tb[AT_THREADS];                                 // pages of the first 64 stages, by wavefront
    __shared__ int32_t vote[AT_WAVES];

    reserve_wide_registers<NB>();
    GRAFT_STAMPS_BEGIN();
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_u = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int kg = wave_u & 1;
    const WorkItem item = xcd_work_item(n_units, n_row_tiles, row_tiles_magic);
    const bool padding = item.unit < 0;
    const int rt = item.row_tile, unit = padding ? 0 : item.unit;             // unit over B * Hkv * n_splits
    const int bg = div31(unit, splits_magic), split = unit - bg * n_splits;
    const int b = div24(bg, n_kv_heads), g = bg - b * n_kv_heads;

    const int n_raw = scalar_load(n_nodes, b), P_raw = scalar_load(prefix_len, b);
    await_setup_args(p);
    if (padding) return;
    const unsigned kv_base = __builtin_amdgcn_readfirstlane(lds_address(&kv[0][0]));
    const int l16 = lane & 15, lg = lane >> 4;
    const int r_tile = rt * S::TILE_ROWS;
    // the queries lie at the end of the ring until they are read
    constexpr unsigned Q_OFF = AT_NBUF * AT_STAGE_BYTES - S::TILE_ROWS * AT_ROW_BYTES;
    constexpr bool Q_OVER_1 = Q_OFF < 2 * AT_STAGE_BYTES;         // they reach into the buffer of stage 1
    request_masks(p, b, Ms, tid, wave_u);
    request_queries<S::TILE_ROWS>(p, b, g, r_tile, kv_base + Q_OFF, lane, wave_u);
    __builtin_amdgcn_sched_barrier(0);
    const SplitRange sr = split_range(p, n_raw, P_raw, split, n_splits, splits_magic);
    const int slots = sr.total - sr.P;           // tree slots that the block table has room for
    const int n_st = sr.st1 - sr.st0;
#ifdef GRAFT_ATTN_STAMPS
    asm volatile("" : : "s"(n_st));
#endif
    GRAFT_STAMP(AT_TS_LENGTHS);

    // page table: lane i holds the page this wavefront moves in stage i of the split, 64 stages at a time
    const int32_t* table = p.block_table + static_cast<size_t>(b) * p.max_pages;
    const int last_tok = sr.total - 1, last_pg = last_tok >> 4;
    auto page_index = [&](int stage) __attribute__((always_inline)) {
        const int pg = (sr.st0 + stage) * (AT_STAGE / GRAFT_PAGE_SIZE) + wave_u;
        return pg < last_pg ? pg : (last_pg < 0 ? 0 : last_pg);
    };
    int32_t first_pages[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) first_pages[u] = scalar_load(table, page_index(u));
    auto load_table = [&](int stage0) __attribute__((always_inline)) {
        int32_t x = table[page_index(stage0 + opaque_lane())];
        asm volatile("" : "+v"(x));              // (waited for here: at its use, the wait would be for the transfers of every stage)
        return x;
    };
    {
        const int lane_now = opaque_lane();
        load_global_to_lds_b32(table + page_index(lane_now), __builtin_amdgcn_readfirstlane(lds_address(Tb)) + 256 * wave_u);
    }
    int32_t pages = 0;
    GRAFT_STAMP(AT_TS_TABLE_REQ);
    const float c_log2 = p.scale_log2e;
    WideState<NB> w;
    auto clear_rows = [&]() __attribute__((always_inline)) {
        static_for<0, 64 * NB>([&](auto k_) {
            GRAFT_CONST(k, k_);
            acc_set<k>(0.0f);
        });
    };
    clear_rows();
#pragma unroll
    for (int rb = 0; rb < NB; ++rb) w.l[rb] = w.negm[rb] = 0.f;
    GRAFT_STAMP(AT_TS_ZEROED);

    // ---- transfers.  A wavefront moves one page a stage: 16 rows of K and of V, four rows (1 KB) per instruction, through a
    //      buffer descriptor that ends with the page's last token (with nothing, past the last page): what lies behind it arrives as
    //      zeros.  Lane (lg, l16) of instruction j fetches a 16-byte chunk of row 4 j + lg: chunk l16 ^ (4 j + lg) of K, 32-byte segment
    //      (l16 / 2) ^ (4 j + lg) % 8 of V.
    const unsigned ts2 = static_cast<unsigned>(p.token_stride) * 2u;
    const unsigned k_chunk = (l16 ^ lg) * 16, v_chunk = ((((l16 >> 1) ^ lg) << 1) | (l16 & 1)) * 16, row_off = lg * ts2;
    const u64 k_head = reinterpret_cast<u64>(p.k) + static_cast<u64>(g * p.head_stride) * 2, v_head = reinterpret_cast<u64>(p.v) + static_cast<u64>(g * p.head_stride) * 2;
    struct PageOf { uintx4 k, v; unsigned lds; };
    auto page_of = [&](int k, int page) __attribute__((always_inline)) {       // what this wavefront moves in stage k
        PageOf d;
        const u64 off = static_cast<u64>(static_cast<unsigned>(page)) * static_cast<u64>(p.page_stride * 2);
        const u64 ka = k_head + off, va = v_head + off;
        const int rows = last_tok - (sr.st0 + k) * AT_STAGE - 16 * wave_u;         // the last token's row in the page
        const unsigned some = static_cast<unsigned>(~(rows >> 31) & ((k - n_st) >> 31));    // all ones where there is something to move
        const unsigned bytes = (static_cast<unsigned>(rows < 15 ? rows : 15) * ts2 + AT_ROW_BYTES) & some;
        d.k = uintx4{static_cast<unsigned>(ka), static_cast<unsigned>(ka >> 32), bytes, BUFFER_WORD3};
        d.v = uintx4{static_cast<unsigned>(va), static_cast<unsigned>(va >> 32), bytes, BUFFER_WORD3};
        d.lds = kv_base + (k & (AT_NBUF - 1)) * AT_STAGE_BYTES + wave_u * 4096;
        return d;
    };
    auto move = [&](const PageOf& d, auto t_) __attribute__((always_inline)) {    // instruction t of 8
        GRAFT_CONST(t, t_);
        constexpr int j = t >> 1;
        // (computed on the spot: eight loop-invariant offsets would take registers that the largest shapes do not have)
        unsigned off;
        asm volatile("v_xor_b32 %0, %1, %2\n\tv_add3_u32 %0, %0, %3, %4"
                     : "=&v"(off)
                     : "i"(t & 1 ? (j & 1) << 7 : j << 6), "v"(t & 1 ? v_chunk : k_chunk), "v"(row_off), "s"(4 * j * ts2));
        buffer_to_lds_b128(t & 1 ? d.v : d.k, off, d.lds + (t & 1) * AT_STAGE * AT_ROW_BYTES + j * 1024);
    };
    auto move_page = [&](int k, int page) __attribute__((always_inline)) {
        const PageOf d = page_of(k, page);
        static_for<0, 8>([&](auto t_) { move(d, t_); });
    };
    if (n_st > 0) move_page(0, first_pages[0]);
    GRAFT_STAMP(AT_TS_STAGE0_REQ);
    if (n_st > 0 && !Q_OVER_1) move_page(1, first_pages[1]);
    // every stage is eight instructions of a wavefront, whatever they move: with eight in flight, all but the newest stage are there
    auto arrive = [&]() __attribute__((always_inline)) {
        GRAFT_SPAN_BEGIN();
        GRAFT_WAIT_VMCNT(AT_LOADS_PER_STAGE);
        GRAFT_SPAN_SPLIT(AT_TS_WAIT_CYCLES);
        lds_barrier();
        GRAFT_SPAN_END(AT_TS_BARRIER_CYCLES);
    };
    GRAFT_MFMA_SETTLE();

    // lane parts of the operand addresses inside a sub-tile
    constexpr unsigned V_OFF = AT_STAGE * AT_ROW_BYTES, SUB = AT_SUB * AT_ROW_BYTES;
    const int v_row = 4 * half + (l16 >> 2);
    const unsigned k_lane = kv_base + l32 * AT_ROW_BYTES + ((l16 >> 1) << 5) + ((half ^ (l16 & 1)) << 4);
    const unsigned v_lane = kv_base + V_OFF + v_row * AT_ROW_BYTES + (((l32 >> 4) ^ (v_row & 7)) << 5) + 8 * (l16 & 3);
    auto sub_base = [&](int k, int visit) __attribute__((always_inline)) {
        return static_cast<unsigned>((k & (AT_NBUF - 1)) * AT_STAGE_BYTES) + S::sub_tile(visit, kg) * SUB;
    };

    bool damaged = false;                        // sums or products that left the range: the exact pass below takes over
    if (n_st > 0) {
        // queries, masks and table are there when only the stages are in flight
        if constexpr (Q_OVER_1) GRAFT_WAIT_VMCNT(AT_LOADS_PER_STAGE);
        else GRAFT_WAIT_VMCNT(2 * AT_LOADS_PER_STAGE);
        lds_barrier();
        GRAFT_STAMP(AT_TS_TABLE_LDS);
        if ((((r_tile + S::TILE_ROWS - 1) * p.g_magic) >> 16) >= sr.n) {       // queries of absent nodes may hold anything: zeros
            for (int x = tid; x < S::TILE_ROWS * AT_ROW_BYTES / 16; x += AT_THREADS)
                if ((((r_tile + x / 16) * p.g_magic) >> 16) >= sr.n) reinterpret_cast<uint4*>(&kv[0][0] + Q_OFF)[x] = uint4{0u, 0u, 0u, 0u};
            lds_barrier();
        }
        pages = Tb[tid];
        uintx4 qd[NB][8];                        // (all reads in flight)
#pragma unroll
        for (int rb = 0; rb < NB; ++rb)
#pragma unroll
            for (int d = 0; d < 8; ++d) qd[rb][d] = __builtin_bit_cast(uintx4, read_k(k_lane + Q_OFF + S::row0(rb, wave_u) * AT_ROW_BYTES, d));
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, NB>([&](auto rb_) {
            GRAFT_CONST(rb, rb_);
            static_for<0, 8>([&](auto d_) {
                GRAFT_CONST(d, d_);
                if constexpr (rb < 2) {
                    static_for<0, 4>([&](auto i_) {
                        GRAFT_CONST(i, i_);
                        acc_set_bits<wide_q<NB>(rb, d) + i>(qd[rb][d][i]);
                    });
                } else {
                    w.q2[d] = __builtin_bit_cast(bf16x8, qd[rb][d]);
                }
            });
        });
        GRAFT_STAMP(AT_TS_Q_DONE);
        if constexpr (Q_OVER_1) {
            lds_barrier();                       // everybody has read
            move_page(1, first_pages[1]);
        }
        GRAFT_STAMP(AT_TS_LOOP);
        GRAFT_STAMP_CYCLES(AT_TS_CYCLES_LOOP);
        arrive();
#ifdef GRAFT_ATTN_STAMPS
        GRAFT_STAMP(AT_TS_STAGE0);
#endif
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            w.k[d] = read_k(k_lane + sub_base(0, 0), d);
            w.v[d] = __builtin_bit_cast(bf16x8, uintx4{0u, 0u, 0u, 0u});
        }
        const PageOf second = page_of(2, first_pages[2]);         // (its transfers go between the first products)
        GRAFT_MFMA_SETTLE();
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) w.p[rb][0] = w.p[rb][1] = uintx4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int v = 0; v < 16; ++v) w.s[S::block(UNITS - 1)][v] = -INFINITY;

        unsigned long long above = 0;
        // PLAIN: not the first stage, and all of it inside the prefix.  Between BAR - 1 and BAR the wavefronts meet: the next stage
        // has landed, and nobody reads the one before this any more, whose buffer the transfers behind it fill.
        auto stage = [&](int k, auto plain_, auto first_) __attribute__((always_inline)) {
            constexpr bool PLAIN = decltype(plain_)::value, FIRST = decltype(first_)::value;
            constexpr int BAR = PLAIN ? 0 : UNITS - 1, SPACE = PLAIN ? 3 : 2;
            PageOf next;
            reserve_wide_registers<NB>();
            static_for<0, UNITS>([&](auto j_) {
                GRAFT_CONST(J, j_);
                if constexpr (J == BAR) arrive();
                const unsigned k_next = k_lane + (J == UNITS - 1 ? sub_base(k + 1, 0) : sub_base(k, 1));
                const unsigned v_next = v_lane + (J < 2 ? sub_base(k, 0) : sub_base(k, 1));
                phase<S, J, true, true, true>(w, c_log2, k_next, v_next, [&](auto i_) __attribute__((always_inline)) {
                    GRAFT_CONST(i, i_);
                    constexpr int at = 16 * (J - BAR) + i;
                    if constexpr (FIRST && J == 0 && i % 2 == 1) move(second, std::integral_constant<int, i / 2>{});
                    if constexpr (at == 0) next = page_of(k + 3, __builtin_amdgcn_readlane(pages, (k + 3) & 63));
                    if constexpr (at > 0 && at % SPACE == 1 % SPACE && at / SPACE < 8) move(next, std::integral_constant<int, (at > 0 ? at / SPACE : 0)>{});
                    if constexpr (J == UNITS - 1 && i == 4) {
                        float lm = w.l[0];
#pragma unroll
                        for (int rb = 1; rb < NB; ++rb) lm = __builtin_fmaxf(lm, w.l[rb]);
                        above = __builtin_amdgcn_ballot_w64(lm > WD_LAZY_SUM);
                        asm volatile("" : "+s"(above));
                    }
                });
                if constexpr (!PLAIN) {
                    constexpr int QB = S::block(J);
                    int t_sub = (sr.st0 + k) * AT_STAGE + S::sub_tile(S::visit(J), kg) * AT_SUB;
                    asm volatile("" : "+s"(t_sub));  // (a condition of its own for every phase: kept for the next one, it goes to a vector register)
                    if (t_sub + AT_SUB > sr.P) {
                        settle(w.s[QB]);
                        const int lz = opaque_lane();
                        mask_scores(w.s[QB], row_window(r_tile + S::row0(QB, wave_u) + (lz & 31), t_sub, sr.P, sr.n, slots, p.R, p.g_magic, Ms), lz >> 5);
                    }
                    // (the sum holds all of the block's earlier units: other blocks' units lie between)
                    const bool unseen = FIRST && S::visit(J) == 0 ? true : pair_sum(w.l[QB]) == 0.f;
                    if (__builtin_amdgcn_ballot_w64(unseen) != 0) {
                        settle(w.s[QB]);
                        const float mx = score_max(w.s[QB]) * c_log2;
                        const bool large = mx > WD_SMALL_SCORE || (mx < 0.f && mx > -INFINITY);
                        w.negm[QB] = unseen ? (large ? -mx : 0.f) : w.negm[QB];
                    }
                }
            });
        };
        int plain_end = (sr.P - sr.st0 * AT_STAGE) / AT_STAGE;                // stages in front of it lie inside the prefix
        plain_end = plain_end < n_st ? plain_end : n_st;
        const auto between = [&](int k) __attribute__((always_inline)) {       // behind stage k - 1, rarely
            if (above != 0) damaged = raise_rows<S>(w) || damaged;
            if (((k + 3) & 63) == 0) {
                pages = load_table(k + 3);
            }
        };
        int k = 1;
        stage(0, std::false_type{}, std::true_type{});
        if (__builtin_expect(above != 0, 0)) between(k);
        for (; k < plain_end;) {
            stage(k, std::true_type{}, std::false_type{});
            ++k;
            if (__builtin_expect((above != 0) | (((k + 3) & 63) == 0), 0)) between(k);
        }
        for (; k < n_st;) {
            stage(k, std::false_type{}, std::false_type{});
            ++k;
            if (__builtin_expect((above != 0) | (((k + 3) & 63) == 0), 0)) between(k);
        }
        reserve_wide_registers<NB>();
        const auto nothing = [](auto) {};
        phase<S, 0, false, true, true>(w, c_log2, 0u, 0u, nothing);
        phase<S, 1, false, false, true>(w, c_log2, 0u, 0u, nothing);
    }
    // Everything has landed: the last stages, or, in a split without a stage, the queries, whose place the exchange below takes.
    GRAFT_WAIT_VMCNT(0);
    GRAFT_MFMA_SETTLE();
    GRAFT_STAMP(AT_TS_LOOP_END);
    GRAFT_STAMP_CYCLES(AT_TS_CYCLES_END);

    // ---- rows whose sum is out of bounds although they see something: once more, with the exact running maximum
    const int lane_end = opaque_lane();
    {
        const int l32 = lane_end & 31, half = lane_end >> 5;
        bool bad = damaged;
        static_for<0, NB>([&](auto rb_) {
            GRAFT_CONST(rb, rb_);
            const float lt = pair_sum(w.l[rb]);
            const int r = r_tile + S::row0(rb, wave_u) + l32;
            bool odd = !(lt >= WD_MIN_SUM && lt < WD_MAX_SUM) && r < p.R && ((r * p.g_magic) >> 16) < sr.n && n_st > 0;
            if (__builtin_amdgcn_ballot_w64(odd) != 0) {          // does it see anything?
                unsigned seen = 0;
                for (int k = 0; k < n_st; ++k)
                    for (int x = 0; x < UNITS / NB; ++x) {
                        const int t_sub = (sr.st0 + k) * AT_STAGE + S::sub_tile(x, kg) * AT_SUB;
                        seen |= row_window(r, t_sub, sr.P, sr.n, slots, p.R, p.g_magic, Ms);
                    }
                bad = bad || __builtin_amdgcn_ballot_w64(odd && seen != 0) != 0;
            }
        });
        if (lane_end == 0) vote[wave_u] = bad ? 1 : 0;
        lds_barrier();                           // (also: nobody reads keys or values any more)
        if (__builtin_expect((vote[0] | vote[1] | vote[2] | vote[3]) != 0, 0)) {
            if (bad) {
                clear_rows();
                static_for<0, NB>([&](auto rb_) {
                    GRAFT_CONST(rb, rb_);
                    w.l[rb] = 0.f;
                    w.negm[rb] = INFINITY;
                });
            }
            move_page(0, first_pages[0]);
            move_page(1, first_pages[1]);
            pages = Tb[wave_u * 64 + lane_end];
            for (int k = 0; k < n_st; ++k) {
                reserve_wide_registers<NB>();
                arrive();
                if (((k + 2) & 63) == 0) pages = load_table(k + 2);
                move_page(k + 2, __builtin_amdgcn_readlane(pages, (k + 2) & 63));
                if (bad) {
                    for (int x = 0; x < 2; ++x) {
                        const int t_sub = (sr.st0 + k) * AT_STAGE + x * AT_SUB;
                        const unsigned at = static_cast<unsigned>((k & (AT_NBUF - 1)) * AT_STAGE_BYTES) + x * SUB;
                        static_for<0, NB>([&](auto rb_) {
                            GRAFT_CONST(rb, rb_);
                            if (!S::SHARED || x == kg) {
                                const bool masked = t_sub + AT_SUB > sr.P;
                                const unsigned win = masked ? row_window(r_tile + S::row0(rb, wave_u) + l32, t_sub, sr.P, sr.n, slots, p.R, p.g_magic, Ms) : ~0u;
                                exact_unit<S, rb>(w, k_lane + at, v_lane + at, masked, win, half, c_log2);
                            }
                        });
                    }
                }
            }
            GRAFT_MFMA_SETTLE();
            GRAFT_WAIT_VMCNT(0);
            lds_barrier();
        }
    }

    // ---- results
    const int lane_out = lane_end;
    const int o32 = lane_out & 31, ohalf = lane_out >> 5;
    const size_t part = ((static_cast<size_t>(b) * n_kv_heads + g) * n_splits + split) * p.R_pad;
    // dims 64 h .. 64 h + 63 of a row block: ov[16 e + v] is dim 64 h + 32 e + 8 (v / 4) + 4 half + v % 4 of row l32
    auto emit = [&](int rb_row0, int h, const float (&ov)[32], float l, float m, bool with_ml) __attribute__((always_inline)) {
        const int r0 = r_tile + rb_row0;
        if (r0 >= p.R) return;
        typedef float floatx2 __attribute__((ext_vector_type(2)));
        typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
        const float inv_l = l > 0.f ? 1.0f / l : 0.f;
        if (n_splits == 1) {
            const int r = r0 + o32, i = (r * p.g_magic) >> 16, hl = r - i * p.G;
            const bool keep = i < sr.n;
            unsigned short* outp = static_cast<unsigned short*>(p.out) +
                ((static_cast<int64_t>(b) * p.K_max + i) * p.Hq + g * p.G + hl) * AT_D + 64 * h + 8 * ohalf;
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    unsigned t[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        t[k] = keep ? pack_bf16(ov[16 * e + 8 * j + 2 * k] * inv_l, ov[16 * e + 8 * j + 2 * k + 1] * inv_l) : 0u;
                    const auto x = __builtin_amdgcn_permlane32_swap(t[0], t[2], false, false);
                    const auto y = __builtin_amdgcn_permlane32_swap(t[1], t[3], false, false);
                    if (r < p.R) *reinterpret_cast<uintx4*>(outp + 32 * e + 16 * j) = uintx4{x[0], y[0], x[1], y[1]};
                }
            return;
        }
        float amax = 0.f;
#pragma unroll
        for (int k = 0; k < 32; ++k) amax = fmaxf(amax, fabsf(ov[k]));
        amax = pair_max(amax);
        int ex = static_cast<int>((__float_as_uint(amax * inv_l) >> 23) & 0xffu);
        ex = ex < 2 ? 126 : (ex > 252 ? 252 : ex);
        const float pow2e = __uint_as_float(static_cast<unsigned>(ex + 1) << 23);      // 2^(ex - 126)
        const float f = inv_l * __uint_as_float(static_cast<unsigned>(253 - ex) << 23);  // 2^-(ex - 126) / l
        unsigned short* op = p.ws_o + (part + r0) * AT_D + h * (AT_D * 16) + 8 * lane_out;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                uintx4 t;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    t[k] = __builtin_bit_cast(unsigned, __builtin_convertvector(
                               floatx2{ov[16 * e + 8 * j + 2 * k] * f, ov[16 * e + 8 * j + 2 * k + 1] * f}, halfx2));
                *reinterpret_cast<uintx4*>(op + 1024 * e + 512 * j) = t;
            }
        if (ohalf == 0) {
            // (sums between one and two, their power of two with the reference: 64 splits' sums of up to 2^26 times values of up to
            //  2^100 would overflow in the merge)
            const int le = static_cast<int>((__float_as_uint(l) >> 23) & 0xffu) - 127, shift = le > -126 && le < 127 ? le : 0;
            float* ml = p.ws_ml + (part + r0 + o32) * 4;
            if (with_ml) *reinterpret_cast<float2*>(ml) =
                float2{l > 0.f ? m + static_cast<float>(shift) : -INFINITY, l * __uint_as_float(static_cast<unsigned>(127 - shift) << 23)};
            ml[2 + h] = pow2e;
        }
    };
    auto own = [&](auto b_, auto h_, float (&ov)[32]) __attribute__((always_inline)) {
        GRAFT_CONST(rb, b_);
        GRAFT_CONST(h, h_);
        static_for<0, 32>([&](auto k_) {
            GRAFT_CONST(k, k_);
            ov[k] = acc_get<wide_o(rb, 2 * h) + k>();
        });
    };
    static_for<0, NB>([&](auto rb_) {
        GRAFT_CONST(rb, rb_);
        w.l[rb] = pair_sum(w.l[rb]);
        if constexpr (!S::SHARED)
            static_for<0, 2>([&](auto h_) {
                GRAFT_CONST(h, h_);
                float ov[32];
                own(rb_, h_, ov);
                emit(S::row0(rb, wave_u), h, ov, w.l[rb], -w.negm[rb], h == 0);
            });
    });
    if constexpr (S::SHARED) {
        // two wavefronts have the same rows and every other sub-tile: each gives half of its dims away and finishes the other
        constexpr int XCH = NB * 32 * 64;         // floats a wavefront gives away
        float* const xch = reinterpret_cast<float*>(&kv[0][0]);
        float* const xml = xch + AT_WAVES * XCH;
        auto give = [&](auto h_) __attribute__((always_inline)) {
            static_for<0, NB>([&](auto rb_) {
                GRAFT_CONST(rb, rb_);
                float ov[32];
                own(rb_, h_, ov);
                float* to = xch + wave_u * XCH + rb * (32 * 64) + 4 * lane_out;
#pragma unroll
                for (int q = 0; q < 8; ++q) *reinterpret_cast<floatx4*>(to + 256 * q) = floatx4{ov[4 * q], ov[4 * q + 1], ov[4 * q + 2], ov[4 * q + 3]};
                if (ohalf == 0) *reinterpret_cast<float2*>(xml + ((wave_u * NB + rb) * 32 + o32) * 2) = float2{-w.negm[rb], w.l[rb]};
            });
        };
        if (kg == 0) give(std::integral_constant<int, 1>{});
        else give(std::integral_constant<int, 0>{});
        lds_barrier();
        auto take = [&](auto h_) __attribute__((always_inline)) {
            GRAFT_CONST(h, h_);
            floatx4 theirs[NB][8];      // (all reads in flight)
            static_for<0, NB>([&](auto rb_) {
                GRAFT_CONST(rb, rb_);
                const float* from = xch + (wave_u ^ 1) * XCH + rb * (32 * 64) + 4 * lane_out;
#pragma unroll
                for (int q = 0; q < 8; ++q) theirs[rb][q] = *reinterpret_cast<const floatx4*>(from + 256 * q);
            });
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, NB>([&](auto rb_) {
                GRAFT_CONST(rb, rb_);
                const float2 other = *reinterpret_cast<const float2*>(xml + (((wave_u ^ 1) * NB + rb) * 32 + o32) * 2);
                const float m0 = w.l[rb] > 0.f ? -w.negm[rb] : -INFINITY, m1 = other.y > 0.f ? other.x : -INFINITY;
                const float mm = fmaxf(m0, m1);
                const float f0 = m0 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m0 - mm), f1 = m1 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m1 - mm);
                float ov[32];
                own(rb_, h_, ov);
#pragma unroll
                for (int q = 0; q < 8; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) ov[4 * q + i] = ov[4 * q + i] * f0 + theirs[rb][q][i] * f1;
                emit(S::row0(rb, wave_u), h, ov, w.l[rb] * f0 + other.y * f1, mm, h == 0);
            });
        };
        if (kg == 0) take(std::integral_constant<int, 0>{});
        else take(std::integral_constant<int, 1>{});
    }
    GRAFT_STAMPS_WRITE(p, n_st);
}

#ifdef GRAFT_WIDE_128
int32_t launch_wide_128(const AttnParams& p, hipStream_t s) {
    const dim3 grid(xcd_grid(static_cast<int64_t>(p.B) * p.Hkv * p.n_splits, p.n_row_tiles));
    launch_attn(tree_attn_wide_128_kernel<2, WIDE_KEYS>, grid, dim3(AT_THREADS), 0, s, p, 1, 1);
    return check_launch();
}
#else
int32_t launch_wide(int32_t tile_rows, const AttnParams& p, hipStream_t s) {
    const dim3 grid(xcd_grid(static_cast<int64_t>(p.B) * p.Hkv * p.n_splits, p.n_row_tiles));
    if (tile_rows == 128) return launch_wide_128(p, s);
    switch (tile_rows) {
        case 192: launch_attn(tree_attn_wide_kernel<3, WIDE_KEYS>, grid, dim3(AT_THREADS), 0, s, p, 1, 1); break;
        case 256: launch_attn(tree_attn_wide_kernel<2, WIDE_ROWS>, grid, dim3(AT_THREADS), 0, s, p, 1, 1); break;
        default: launch_attn(tree_attn_wide_kernel<3, WIDE_ROWS>, grid, dim3(AT_THREADS), 0, s, p, 1, 1); break;   // 384
    }
    return check_launch();
}
#endif

}  // namespace graft
