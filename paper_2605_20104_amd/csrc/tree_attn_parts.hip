// graft_tree_attn, direct path: fp32 storage with the products on the 16-bit matrix cores.
//
// The shape is that of tree_attn_direct_kernel with two row blocks and one row group: a workgroup has 32 query rows, its eight
// wavefronts take every eighth tile of 32 keys each, without a barrier, and merge through LDS at the end.
//   why   : v_mfma_f32_16x16x4_f32 binds that kernel (8192 of a step's 8200 cycles), at a sixteenth of the 16-bit rate.  Here a number is
//           the sum of 16-bit ones, and a product the sum of theirs: each of them exact, their sums fp32.  Mean relative error against 64
//           bits over seven shapes of 200 to 700 tokens 4.2e-7 with fp32 products, 2.7e-7 so, smaller in every one.
//   S     : queries and keys are two fp16 numbers, h the nearest one and m the nearest one to what h leaves: 23 bits.  A product is h h +
//           h m + m h (m m is below 2^-24 of it), 24 roundings a score where four numbers at a time took 32.  fp16 ends at 2^16 and
//           loses bits below 2^-14, so numbers are taken times powers of two (exact): a row's largest query is brought to 2^8, and
//           the keys of a tile are taken as they are or, where they are small, with the largest at 2^8.
//           What is lost even so, up to 2^-25 of a scaled number, counts where small operands stand beside large ones that meet
//           zeros.  So a wavefront keeps the smallest factor and the largest key of its tiles, and behind the last of them has for
//           every row a bound of it: scale * 2^-25 (|q| / factor of the keys + sqrt(D) * largest key / factor of the queries), the
//           2-norm and not the sum of |q|, as the errors of D numbers are independent.  It may be 2^-22 (of a weight, as much as the
//           rounding of an exponent of 4) or that part of the row's largest score (at least as far from zero as its reference is, or 16
//           less: a reference is kept that long), which fp32 sums of D products are off by too.
//   O     : probabilities and values are three bf16 numbers whose sum they are, eight bits each, and a product six of the nine (the rest is
//           below 2^-23 of it): the exponents are those of fp32, so there is nothing to scale and nothing to lose (above 2^-133, where
//           bf16 numbers end), whatever the values of a dim have been before and whatever other rows see.  (Two fp16 numbers with a factor a dim from the wavefront's
//           first tile: 4.0 us a step, and wrong results behind values of another size, by 7e-3 and without end.)
//   beyond: what fp16 does not hold (keys past 65504, infinities, NaN) makes sums infinite or NaN.  Such a wavefront, and one
//           with a row past the bound above, takes its tiles once more with v_mfma_f32_32x32x2_f32 on the same registers, and keys
//           with values that are not finite kept out of the product.
//   K     : straight from memory to a wavefront-private piece of LDS, 16-byte chunks XOR-swizzled with the row; a lane reads
//           8 dims of its key and splits them as it goes.
//   V     : straight to registers.  Lane (half, l32) holds keys 8 (v / 4) + 4 half + v % 4, v < 16, in D / 32 dims from l32 D / 32
//           on, which is the A operand of O^T = V^T P^T for each of these dims without an exchange between lanes.
//   S, P  : a lane has row l32 and the same 16 keys of the scores.
//   order : the products of a step and the split of the next one's numbers take turns (sched_group_barrier): without, the wavefront
//           waits for LDS and the matrix cores in turn (bf16 parts, three a number, 6.3 us a step without and 6.0 with).
//
// Measured (MI355X), fp32 products / this kernel.  A step, 256 keys of a row tile, 256 workgroups whose keys come from the caches: D = 128
// 7.69 / 5.05 us, D = 64 4.66 / 2.95.  us a call: 1 sequence of 2048 keys, 40 x 32 heads on 8, 22.6 / 18.1; 8192, 64 x 40 on 8, 96.8 / 65.5; 4 of
// 1024, 40 x 32 on 8, 41.3 / 25.4; D = 64, 2 of 5000, 60 x 16 on 4, 31.9 / 22.5.  Keys of 0.05, which are scaled: 22.0 / 20.1, 96.5 / 71.8,
// 41.4 / 29.9, 30.7 / 25.2.
// Tried and dropped: three bf16 numbers for queries and keys too (20.2 us instead of 18.1, 78.2 instead of 65.5); the bf16 split by
// v_dot2_f32_bf16, three and a half instructions a number instead of five and a half but at a lower rate (19.4, 72); the fp16 split by
// v_fma_mixlo_f16 and its high half (two instructions a number with the factor, but at half the rate).
#include "attn_direct.h"

namespace graft {

constexpr int PT_TK = 32;                       // keys of a tile
constexpr int PT_ROWS = 32;                     // query rows of a workgroup
constexpr int PT_TOP = 8;                       // largest queries of a row, and keys of a tile that is scaled, are brought to 2^8 .. 2^9
constexpr float PT_KEY_MIN = 0.25f;             // a tile whose half keys (a lane's dims of one) all reach it is taken as it is
constexpr float PT_LOST = 0x1p-22f;             // what lost bits may move a score by, or that part of the row's reference

typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));

// Eight numbers of a lane as two operands: the nearest fp16 numbers and those of what they leave.  Two instructions a number, all
// of them at the full rate; v_fma_mixlo_f16 and its high half, two a number with a factor, run at half of it.
struct Parts { half8_t h, m; };
__device__ __forceinline__ Parts split8(const float (&x)[8]) {
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    Parts r;
    float minus_one = -1.f;
    asm("" : "+s"(minus_one));                   // (x - h as one v_fma_mix_f32; the compiler takes a plain difference apart)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        half2_t h = __builtin_convertvector(floatx2{x[2 * j], x[2 * j + 1]}, half2_t);
        asm("" : "+v"(h));                       // (the pair in one register: both halves are read from there)
        const half2_t m = __builtin_convertvector(floatx2{__builtin_fmaf(static_cast<float>(h[0]), minus_one, x[2 * j]),
                                                          __builtin_fmaf(static_cast<float>(h[1]), minus_one, x[2 * j + 1])}, half2_t);
        r.h[2 * j] = h[0];
        r.h[2 * j + 1] = h[1];
        r.m[2 * j] = m[0];
        r.m[2 * j + 1] = m[1];
    }
    return r;
}
template <bool SCALED> __device__ __forceinline__ Parts split8(const float (&x)[8], float c) {
    float y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = SCALED ? x[i] * c : x[i];
    return split8(y);
}
// Largest and smallest numbers of an operand, pair by pair.  (Of the fp16 ones, which are there for the products anyway: a maximum over the
// fp32 ones kept those in registers, 72 of which went to memory.)
__device__ __forceinline__ void widest(half2_t& hi, half2_t& lo, const half8_t& h) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const half2_t x{h[2 * i], h[2 * i + 1]};
        hi = __builtin_elementwise_maximum(hi, x);
        lo = __builtin_elementwise_minimum(lo, x);
    }
}
__device__ __forceinline__ float max_abs(float acc, const float (&x)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = __builtin_fmaxf(acc, __builtin_fabsf(x[i]));
    return acc;
}
// Eight numbers of a lane as three bf16 operands, whose sum they are: eight bits of a number, eight of what they leave, and what those
// leave.  (Infinities leave NaN.)  NEAREST: rounded, not cut off, which makes what a product leaves out a quarter and of either sign, but
// takes v_cvt_pk_bf16_f32 where a v_perm_b32 does.
struct Thirds { bf8_t h, m, l; };
template <bool NEAREST> __device__ __forceinline__ Thirds split_exactly(const float (&x)[8]) {
    uintx4 h, m, l;
    const auto upper = [](unsigned v) __attribute__((always_inline)) { return __uint_as_float(v & 0xffff0000u); };
    const auto uppers = [](float a, float b) __attribute__((always_inline)) {
        return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
    };
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float a = x[2 * j], b = x[2 * j + 1];
        float a1, b1, a2, b2;
        if constexpr (NEAREST) {
            h[j] = pack_bf16(a, b);
            a1 = a - __uint_as_float(h[j] << 16), b1 = b - upper(h[j]);
            m[j] = pack_bf16(a1, b1);
            a2 = a1 - __uint_as_float(m[j] << 16), b2 = b1 - upper(m[j]);
        } else {
            h[j] = uppers(a, b);
            a1 = a - upper(__float_as_uint(a)), b1 = b - upper(__float_as_uint(b));
            m[j] = uppers(a1, b1);
            a2 = a1 - upper(__float_as_uint(a1)), b2 = b1 - upper(__float_as_uint(b1));
        }
        l[j] = uppers(a2, b2);
    }
    return Thirds{__builtin_bit_cast(bf8_t, h), __builtin_bit_cast(bf8_t, m), __builtin_bit_cast(bf8_t, l)};
}
__device__ __forceinline__ floatx16 mfma_f16(const half8_t& a, const half8_t& b, const floatx16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx16 mfma_bf16(const bf8_t& a, const bf8_t& b, const floatx16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// The power of two that takes a largest magnitude to 2^PT_TOP .. 2^(PT_TOP + 1); 2^PT_TOP for zero and for what is not finite.
__device__ __forceinline__ int scale_exponent(float largest) {
    const int e = static_cast<int>((__float_as_uint(largest) >> 23) & 0xffu);
    const int s = PT_TOP - (e - 127);
    return e == 0 || e == 255 ? PT_TOP : (s > 100 ? 100 : (s < -100 ? -100 : s));
}
__device__ __forceinline__ float pow2(int e) { return __uint_as_float(static_cast<unsigned>(e + 127) << 23); }

template <int D>
__global__ __launch_bounds__(DR_THREADS, 2) void tree_attn_parts_kernel(GRAFT_ATTN_ARGS) {
    constexpr int ROW = D * 4, CPR = ROW / 16, RPI = 1024 / ROW;   // bytes and chunks of a row, rows of a 1 KB transfer
    constexpr int STEPS = D / 16, NJ = D / 32;                    // of the first product; dims of a lane's values
    constexpr int KEYS_BYTES = PT_TK * ROW, NK = KEYS_BYTES / 1024;
    constexpr int KG = DR_WAVES, PAGES = PT_TK / GRAFT_PAGE_SIZE, TPR = 64 / PAGES;
    constexpr int PITCH = D + 4;
    typedef float floatj __attribute__((ext_vector_type(NJ)));
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    unsigned char* const Qs = lds + DR_MASK_BYTES;                 // [part][step][lane] operands, then keys
    float* const merge_lds = reinterpret_cast<float*>(Qs);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const WorkItem item = xcd_work_item(n_units, n_row_tiles, row_tiles_magic);
    const bool padding = item.unit < 0;
    const int rt = item.row_tile, unit = padding ? 0 : item.unit;
    const int bg = div31(unit, splits_magic), split = unit - bg * n_splits;
    const int b = div24(bg, n_kv_heads), g = bg - b * n_kv_heads;

    const int b_lane = per_lane(b);
    const int n_lane = n_nodes[b_lane], P_lane = prefix_len[b_lane];
    await_setup_args(p);
    if (padding) return;
    const int32_t* table = p.block_table + static_cast<size_t>(b) * p.max_pages;
    const int per_full = div31((p.max_pages + PAGES - 1) / PAGES + n_splits - 1, splits_magic);
    int tb = 0;
    {
        const int pg = (split * per_full + wave + KG * (lane / PAGES)) * PAGES + lane % PAGES;
        tb = table[pg < p.max_pages ? pg : p.max_pages - 1];
    }
    const int r_base = rt * PT_ROWS;
    const auto row_node = [&](int r) __attribute__((always_inline)) { return ((r < p.R ? r : 0) * p.g_magic) >> 16; };     // rows past R read row 0
    const auto query_row = [&](int x) __attribute__((always_inline)) {         // of lane x
        const int r = r_base + (x & 31), node = row_node(r);
        return static_cast<const float*>(p.q) +
            ((static_cast<size_t>(b) * p.K_max + node) * p.Hq + (g * p.G + ((r < p.R ? r : 0) - node * p.G))) * D + 8 * (x >> 5);
    };
    // The lane index, for what is rarely needed or cheap: taken from here it is computed on the spot.  Registers are short, and whatever
    // stays in one across the loop sends something else to memory.
    const auto lane_now = [&]() __attribute__((always_inline)) { return per_lane(lane); };
    floatx4 q0{}, q1{};
    if (wave < STEPS) {
        const float* q_row = query_row(lane) + 16 * wave;
        q0 = *reinterpret_cast<const floatx4*>(q_row);
        q1 = *reinterpret_cast<const floatx4*>(q_row + 4);
    }
    unsigned mask_word = 0;
    if (tid < p.K_max * 4) mask_word = reinterpret_cast<const unsigned*>(p.mask + static_cast<size_t>(b) * p.K_max * GRAFT_MASK_WORDS)[tid];

    __builtin_amdgcn_sched_barrier(0);
    const int n_raw = __builtin_amdgcn_readfirstlane(n_lane), P_raw = __builtin_amdgcn_readfirstlane(P_lane);
    int n = n_raw;
    if (n < 1 || n > p.K_max) n = 0;
    const int cap = p.max_pages * GRAFT_PAGE_SIZE;
    int P = P_raw;
    P = P < 0 ? 0 : (P > cap ? cap : P);
    const int total = n ? ((P + n) < cap ? (P + n) : cap) : 0;
    const int n_tiles = (total + PT_TK - 1) / PT_TK;
    const int per_split = div31(n_tiles + n_splits - 1, splits_magic);
    const int tile0 = split * per_split;
    const int tile1 = (tile0 + per_split) < n_tiles ? (tile0 + per_split) : n_tiles;
    const int first = tile0 + wave;
    const bool rows_live = ((r_base * p.g_magic) >> 16) < n && r_base < p.R;
    const int count = (rows_live && first < tile1) ? (tile1 - first + KG - 1) / KG : 0;

    float m, l;
    int k_exp = 0;                               // keys of a tile are taken times 2 to this,
    int k_low = 127;                             // least of these exponents
    float k_top = 0.f;                           // largest key of a lane
    floatx16 o[NJ];                              // o[j][u]: dim NJ (8 (u / 4) + 4 half + u % 4) + j of row l32
    auto clear_rows = [&]() __attribute__((always_inline)) {
        m = -INFINITY;
        l = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) o[j] = floatx16{};
    };

    const int last = total - 1, last_pg = last >> 4;
    const char* kc = static_cast<const char*>(p.k) + static_cast<int64_t>(g) * p.head_stride * 4;
    const char* vc = static_cast<const char*>(p.v) + static_cast<int64_t>(g) * p.head_stride * 4;
    const unsigned ts = static_cast<unsigned>(p.token_stride) * 4u;
    // (a wavefront's last tile first: the one tile that can reach past the end is only ever the first of a wavefront, and
    // loads inside the loop need no branch)
    auto tile_at = [&](int it) __attribute__((always_inline)) { return first + KG * (it == 0 ? count - 1 : it - 1); };
    auto load_table = [&](int it) __attribute__((always_inline)) {
        const int pg = tile_at(it + lane / PAGES) * PAGES + lane % PAGES;
        tb = table[pg < last_pg ? pg : last_pg];
    };
    const bool in_order = count <= TPR && (n_splits == 1 || per_split == per_full);
    if (in_order) {
        const int tile = tile_at(0), over = last_pg - tile * PAGES;   // a page past the last one repeats it
        const int at = (count - 1) * PAGES + (over < PAGES - 1 ? over : PAGES - 1);
        const int entry = __builtin_amdgcn_readlane(tb, at & 63);
        tb = lane > at ? entry : tb;
    } else if (count > 0) {
        load_table(0);
        asm volatile("" : "+v"(tb));             // (waited for here: behind the join it would be for everything requested)
    }
    auto table_slot = [&](int it) __attribute__((always_inline)) {
        return in_order ? (it == 0 ? count - 1 : it - 1) & (TPR - 1) : it & (TPR - 1);
    };
    auto page_base = [&](int it, int c) __attribute__((always_inline)) {
        return static_cast<int64_t>(__builtin_amdgcn_readlane(tb, table_slot(it) * PAGES + c)) * p.page_stride * 4;
    };
    // ---- keys.  Transfer j brings rows j RPI ..: slot s of a row holds its chunk s ^ (row & 15)
    unsigned char* const Ks0 = Qs + 2 * STEPS * 1024;
    unsigned char* const Ks = Ks0 + wave * KEYS_BYTES;
    // (lane x brings row x / CPR of a transfer's, and of the chunks the one whose place is x % CPR)
    const auto key_chunk = [&](int x, int j) __attribute__((always_inline)) {
        return static_cast<unsigned>(((x % CPR) ^ (x / CPR) ^ (j * RPI & 15)) * 16);
    };
    const unsigned ks_lds = __builtin_amdgcn_readfirstlane(lds_offset(Ks));
    const auto transfer = [&](const char* base, unsigned off, int j) __attribute__((always_inline)) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(ks_lds + j * 1024), "v"(off), "s"(base) : "memory");
    };
    auto load_keys = [&](int it) __attribute__((always_inline)) {
        const int x = lane_now();
        const unsigned off = x / CPR * ts;
#pragma unroll
        for (int j = 0; j < NK; ++j)
            transfer(kc + page_base(it, j * RPI / 16) + static_cast<int64_t>(j * RPI % 16) * ts, off + key_chunk(x, j), j);
    };
    // ---- values: value v is key 8 (v / 4) + 4 half + v % 4
    floatj vt[16];
    auto load_values = [&](int it) __attribute__((always_inline)) {
        const int x = lane_now();
        const unsigned off = 4 * (x >> 5) * ts + (x & 31) * (NJ * 4);
#pragma unroll
        for (int v = 0; v < 16; ++v)
            vt[v] = *reinterpret_cast<const floatj*>(vc + page_base(it, v >> 3) + static_cast<int64_t>(8 * (v >> 2 & 1) + (v & 3)) * ts + off);
    };
    // a tile that may reach past the end: keys past the last token read the last token again (its probability there is zero)
    auto row_off = [&](int it, int page, int k) __attribute__((always_inline)) {
        const int t_page = tile_at(it) * PT_TK + 16 * page;
        const int lim = last - (t_page < last ? t_page : (last & ~15));
        return static_cast<unsigned>(k < lim ? k : lim) * ts;
    };
    auto load_clamped = [&](int it) __attribute__((always_inline)) {
        const int x = lane_now();
#pragma unroll
        for (int j = 0; j < NK; ++j)
            transfer(kc + page_base(it, j * RPI / 16), row_off(it, j * RPI / 16, j * RPI % 16 + x / CPR) + key_chunk(x, j), j);
#pragma unroll
        for (int v = 0; v < 16; ++v)
            vt[v] = *reinterpret_cast<const floatj*>(vc + page_base(it, v >> 3) +
                (row_off(it, v >> 3, 8 * (v >> 2 & 1) + 4 * (x >> 5) + (v & 3)) + (x & 31) * (NJ * 4)));
    };
    const float sc = p.scale_log2e;
    if (count > 0) load_clamped(0);
    // queries and masks to LDS
    if (tid < p.K_max * 4) reinterpret_cast<unsigned*>(lds)[tid] = mask_word;
    // (a row's largest query: every wavefront has its step's)
    float* const q_top = reinterpret_cast<float*>(Ks0 + DR_WAVES * KEYS_BYTES);
    const float x[8] = {q0[0], q0[1], q0[2], q0[3], q1[0], q1[1], q1[2], q1[3]};
    if (wave < STEPS) {
        q_top[wave * 32 + l32] = row_max<32>(max_abs(0.f, x));
    }
    lds_only_barrier();
    float q_max = 0.f;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) q_max = __builtin_fmaxf(q_max, q_top[s * 32 + l32]);
    const int q_exp = scale_exponent(q_max);
    float* const q_squares = q_top + STEPS * 32;                   // sums of the scaled queries' squares, likewise
    if (wave < STEPS) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) t += (x[i] * pow2(q_exp)) * (x[i] * pow2(q_exp));
        q_squares[wave * 32 + l32] = row_sum<32>(t);
        const Parts q = split8<true>(x, pow2(q_exp));
        *reinterpret_cast<half8_t*>(Qs + wave * 1024 + lane * 16) = q.h;
        *reinterpret_cast<half8_t*>(Qs + (STEPS + wave) * 1024 + lane * 16) = q.m;
    }
    lds_only_barrier();
    const float row_scale = sc * pow2(-q_exp);
    float s_scale = row_scale * pow2(-k_exp);
    const uintx4* mask_lds = reinterpret_cast<const uintx4*>(lds);
    // (dims 16 s + 8 half .. of key l32: chunks 4 s + 2 half + i at that ^ (l32 & 15).  The lane's part of the address is taken anew for
    //  every tile: eight loop-invariant addresses would take registers that are short here)
    unsigned k_addr = lds_offset(Ks) + l32 * ROW + ((2 * half) ^ (l32 & 15)) * 16;
    const auto key_dims = [&](int s, float (&x)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const floatx4 c = *reinterpret_cast<const floatx4 __attribute__((address_space(3)))*>(
                static_cast<size_t>((k_addr ^ static_cast<unsigned>((4 * (s & 3) + i) * 16)) + (s >> 2) * 256));
#pragma unroll
            for (int t = 0; t < 4; ++t) x[4 * i + t] = c[t];
        }
    };
    const auto query_dims = [&](int d) __attribute__((always_inline)) {
        const unsigned char* at = Qs + d * 1024 + lane * 16;
        return Parts{*reinterpret_cast<const half8_t*>(at), *reinterpret_cast<const half8_t*>(at + STEPS * 1024)};
    };
    // One tile; more: the next one is requested.  (A condition and not a second copy of the step: with a few tiles a wavefront the
    // instructions are cold, and fewer of them are the faster code.)
    auto step = [&](int it, bool more, auto careful_) __attribute__((always_inline)) {
        constexpr bool careful = decltype(careful_)::value;
        const int t0 = tile_at(it) * PT_TK;
        floatx16 s;
        asm volatile("" : "+v"(k_addr));
        asm volatile("s_waitcnt vmcnt(16)" ::: "memory");          // the tile's keys, its 16 loads of values may be on their way
        if constexpr (careful) {
            s = floatx16{};
            const float* q_row = query_row(lane_now());
#pragma unroll 1
            for (int d = 0; d < STEPS; ++d) {
                float x[8];
                key_dims(d, x);
                const floatx4 a = *reinterpret_cast<const floatx4*>(q_row + 16 * d), c = *reinterpret_cast<const floatx4*>(q_row + 16 * d + 4);
#pragma unroll
                for (int i = 0; i < 8; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], i < 4 ? a[i & 3] : c[i & 3], s, 0, 0, 0);
            }
        } else {
            // a step's three products beside the next one's split and the reads of the one after it
            const auto products = [&](auto scaled_) __attribute__((always_inline)) {
                constexpr bool SCALED = decltype(scaled_)::value;
                const float c = pow2(k_exp);
                half2_t hi{}, lo{};
                s = floatx16{};
                float x[2][8];
                Parts ks[2], qs[2];
                key_dims(0, x[0]);
                qs[0] = query_dims(0);
                key_dims(1, x[1]);
                ks[0] = split8<SCALED>(x[0], c);
#pragma unroll
                for (int d = 0; d < STEPS; ++d) {
                    const Parts &k = ks[d & 1], &q = qs[d & 1];
                    if (d + 1 < STEPS) qs[(d + 1) & 1] = query_dims(d + 1);
                    if (d + 2 < STEPS) key_dims(d + 2, x[d & 1]);
                    widest(hi, lo, k.h);
                    if (d + 1 < STEPS) ks[(d + 1) & 1] = split8<SCALED>(x[(d + 1) & 1], c);
                    s = mfma_f16(k.m, q.h, s);
                    s = mfma_f16(k.h, q.m, s);
                    s = mfma_f16(k.h, q.h, s);
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
                    }
                }
                const half2_t both = __builtin_elementwise_maximum(hi, -lo);
                const float top = static_cast<float>(__builtin_elementwise_maximum(both[0], both[1])) * (SCALED ? pow2(-k_exp) : 1.f);
                k_top = __builtin_elementwise_maximum(k_top, top);
                return __builtin_amdgcn_ballot_w64(top < PT_KEY_MIN) == 0;
            };
            if (__builtin_expect(!(k_exp == 0 && products(std::false_type{})), 0)) {
                float t = 0.f, x[8];
#pragma unroll 1
                for (int d = 0; d < STEPS; ++d) {
                    key_dims(d, x);
                    t = max_abs(t, x);
                }
                t = wave_max_f32(t);
                const int e = t >= 0x1p9f && t < 0x1p15f ? 0 : scale_exponent(t);
                if (e != 0 || k_exp != 0) {
                    k_exp = e;                                     // (zero: the next tile is tried as it is again)
                    s_scale = row_scale * pow2(-k_exp);
                    (void)products(std::true_type{});
                }
            }
            k_low = k_exp < k_low ? k_exp : k_low;
        }
        unsigned odd = 0;                                          // keys with an infinite or NaN value
        if constexpr (careful) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                bool bad = false;
#pragma unroll
                for (int j = 0; j < NJ; ++j) bad = bad || !__builtin_isfinite(vt[v][j]);
                odd |= bad ? 1u << (8 * (v >> 2) + (v & 3)) : 0u;
            }
            odd <<= 4 * half;
#pragma unroll
            for (int x = 32; x >= 1; x >>= 1) odd |= __shfl_xor(odd, x);
            odd = __builtin_amdgcn_readfirstlane(odd);
        }
        if (__builtin_expect(t0 + PT_TK > P, 0)) {
            const int x = lane_now();
            const uintx4 words = mask_lds[row_node(r_base + (x & 31))];
            const unsigned win = visible_window(t0 - P, total - P, [&](int k) {
                return k == 0 ? words[0] : (k == 1 ? words[1] : (k == 2 ? words[2] : words[3]));
            }) >> (4 * (x >> 5));
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = keep_visible(s[v], win, 8 * (v >> 2) + (v & 3));
        }
        float mx = s[0];                                           // (a row with a NaN among its scores is NaN either way)
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = __builtin_elementwise_maximum(mx, s[v]);
        const float f = careful ? sc : s_scale;
        mx *= f;
        // (rare) a row without a reference, or one that outgrew it: raise it to the maximum seen
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(mx > m + (careful ? 0.f : DR_LAZY_LOG2)) != 0, 0)) {
            const float mn = fmaxf(m, row_max<32>(mx));
            const float a = mn == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m - mn);
            m = mn;
            l *= a;
#pragma unroll
            for (int j = 0; j < NJ; ++j) o[j] *= a;
        }
        const float neg = m == -INFINITY ? 0.f : -m;
        float sum = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[v], f, neg));
            sum += s[v];
        }
        l += sum;
        // the values of such a key leave the product and are added to the rows that see it
        for (unsigned left = odd; careful && left != 0; left &= left - 1) {
            const int key = __builtin_ctz(left), page = key >> 4, at = (key >> 3) * 4 + (key & 3), group = key >> 2 & 1;
            const char* vrow = vc + page_base(it, page) + row_off(it, page, key & 15);
            float pk = s[0];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                pk = at == v ? s[v] : pk;
                if (half == group && at == v) vt[v] = floatj{};
            }
            pk = __shfl(pk, 32 * group + l32);
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                if (pk != 0.f) {
                    const floatj x = *reinterpret_cast<const floatj*>(vrow + (8 * (u >> 2) + 4 * half + (u & 3)) * (NJ * 4));
#pragma unroll
                    for (int j = 0; j < NJ; ++j) o[j][u] += x[j] * pk;
                }
                asm volatile("" ::: "memory");                     // (one load at a time: registers are short here)
            }
        }
        if constexpr (careful) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
#pragma unroll
                for (int j = 0; j < NJ; ++j) o[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(vt[v][j], s[v], o[j], 0, 0, 0);
        } else {
            // The next tile's keys are requested when this one's values are there (what waits for values counts none of the
            // transfers) and its keys have long been read.
#pragma unroll
            for (int v = 0; v < 16; ++v) asm volatile("" : "+v"(vt[v]) : : "memory");
            if (more) load_keys(it + 1);
            const auto probabilities = [&](int kk) __attribute__((always_inline)) {
                float x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = s[8 * kk + i];
                return split_exactly<true>(x);
            };
            const auto values = [&](int kk, int j) __attribute__((always_inline)) {
                float x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = vt[8 * kk + i][j];
                return split_exactly<false>(x);
            };
            // six products of an accumulator beside the split of the next dim's values
            Thirds pp[2], v[2];
            pp[0] = probabilities(0);
            v[0] = values(0, 0);
#pragma unroll
            for (int u = 0; u < 2 * NJ; ++u) {                     // keys 16 (u / NJ) .., dim u % NJ
                const int kk = u / NJ, j = u % NJ, kk1 = (u + 1) / NJ, j1 = (u + 1) % NJ;
                const Thirds &a = v[u & 1], &q = pp[kk];
                if (u == NJ - 2) pp[1] = probabilities(1);
                if (u + 1 < 2 * NJ) v[(u + 1) & 1] = values(kk1, j1);
                o[j] = mfma_bf16(a.l, q.h, o[j]);
                o[j] = mfma_bf16(a.m, q.m, o[j]);
                o[j] = mfma_bf16(a.h, q.l, o[j]);
                o[j] = mfma_bf16(a.m, q.h, o[j]);
                o[j] = mfma_bf16(a.h, q.m, o[j]);
                o[j] = mfma_bf16(a.h, q.h, o[j]);
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
                }
            }
        }
        if (more) load_values(it + 1);
    };
    clear_rows();
    // chunks of the tiles that one table register covers
    for (int it = 0; it < count;) {
        const int end = it + TPR < count ? it + TPR : count;
        if (it > 0) {
            load_table(it);
            load_clamped(it);
        }
        for (; it < end; ++it) step(it, it + 1 < end, std::false_type{});
    }
    {
        float t = 0.f;                                             // two sums per instruction, NaN is kept
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int u = 0; u < 16; ++u) t = __builtin_elementwise_maximum(t, __builtin_fabsf(o[j][u]));
        float squares = 0.f;
#pragma unroll
        for (int d = 0; d < STEPS; ++d) squares += q_squares[d * 32 + l32];
        const float lost = __builtin_amdgcn_ldexpf(__builtin_amdgcn_sqrtf(squares), -25 - k_low) +
                           __builtin_sqrtf(static_cast<float>(D)) * 0x1p-25f * wave_max_f32(k_top);
        const bool fine = t < INFINITY && __builtin_fabsf(row_scale) * lost <= PT_LOST * __builtin_fmaxf(1.f, __builtin_fmaxf(m, -m - DR_LAZY_LOG2));
        const bool odd = !fine && row_node(r_base + (lane_now() & 31)) < n;              // (queries of absent nodes may be anything)
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd) != 0, 0)) {
            clear_rows();
            for (int it = 0; it < count; ++it) {
                if (!in_order && it % TPR == 0) load_table(it);
                load_clamped(it);
                step(it, false, std::true_type{});
            }
        }
    }
    l = row_sum<32>(l);
    // ---- results: the eight wavefronts' rows, merged through LDS
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");               // (nothing is on its way by now: so it stays, whatever the loop becomes)
    __syncthreads();                                               // nobody reads keys or queries any more
    float* ml_lds = merge_lds + DR_WAVES * PT_ROWS * PITCH;
    {
        float* row = merge_lds + (wave * PT_ROWS + l32) * PITCH;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            floatj x;
#pragma unroll
            for (int j = 0; j < NJ; ++j) x[j] = o[j][u];
            *reinterpret_cast<floatj*>(row + (8 * (u >> 2) + 4 * half + (u & 3)) * NJ) = x;
        }
        if (half == 0) *reinterpret_cast<float2*>(ml_lds + 2 * (wave * PT_ROWS + l32)) = float2{m, l};
    }
    __syncthreads();
    const size_t part = ((static_cast<size_t>(b) * n_kv_heads + g) * n_splits + split) * p.R_pad;
    merge_key_groups<float, D, KG>(p, merge_lds, ml_lds, PT_ROWS, r_base, tid, b, g, n, n_splits, part);
}

// LDS of a workgroup: masks, then queries and keys, or the merge
static constexpr size_t parts_lds_bytes(int32_t D) {
    const size_t loop = 2 * (D / 16) * 1024 + static_cast<size_t>(DR_WAVES) * PT_TK * D * 4 + 2 * (D / 16) * 32 * sizeof(float);
    const size_t merge = static_cast<size_t>(DR_WAVES) * PT_ROWS * (D + 4 + 2) * sizeof(float);
    return DR_MASK_BYTES + (loop > merge ? loop : merge);
}
static_assert(parts_lds_bytes(128) <= DR_LDS_BYTES, "one workgroup a compute unit");

int32_t launch_parts(const DirectPlan& pl, const AttnParams& p, int32_t D, hipStream_t s) {
    const unsigned lds = static_cast<unsigned>(parts_lds_bytes(D));
    return D == 64 ? launch_pieces<float, 64, tree_attn_parts_kernel<64>>(pl, p, lds, s) : launch_pieces<float, 128, tree_attn_parts_kernel<128>>(pl, p, lds, s);
}

}  // namespace graft
