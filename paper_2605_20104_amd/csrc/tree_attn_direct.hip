// graft_tree_attn, direct path: fp32 storage (any head size; the longer sequences take tree_attn_parts.hip), bf16 with D = 64, and bf16
// with D = 128 where the keys are few.  Plans and launches of both.
//
// A wavefront owns its keys: the wavefronts of a workgroup split a key range between them (kg
// key groups), as well as the query rows (rg row groups of MB 16-row blocks), walk their tiles (32
// keys in bf16, 16 in fp32) without a barrier and merge at the end through LDS, so that a short
// prefix is spread over the chip with few or no partial results in memory.
//   fp32 : v_mfma_f32_16x16x4_f32 (full fp32 products and sums, 32 cycles each).  The kernel is
//          bound by them: 64 (D = 128) or 32 (D = 64) per 16 keys and 16 rows.
//   bf16 : v_mfma_f32_16x16x32_bf16, and with D = 64 and two or four row blocks v_mfma_f32_32x32x16_bf16, on raw
//          Q and K (exact products, fp32 sums); the softmax scale is applied in fp32.  With D = 64 probabilities enter the second product whole, as the sum of
//          three bf16 numbers (two, 17 bits, put the results further from a 64-bit reference), with
//          D = 128 rounded to one, as on the path this stands in for.  Bound by the vector ALUs (exp2 and the
//          packing of probabilities).
// Operand layouts of blocks of 16 rows (lane = 16 lg + l16); those of 32 rows stand at DirectOps<__bf16, D, 32>.  First product: S^T = K Q^T, A = K (key l16), B = Q^T
// (row l16), so a lane gets 4 keys (4 lg + i) of one row, and these are the B operand of the
// second product O^T = V^T P^T without any exchange between lanes: its contraction index runs
// over the same keys (16 c + 4 lg + i).  Its A operand wants one dim of those keys per lane: in
// fp32 a lane loads four consecutive dims of a key and uses one per MFMA (the assignment of dims
// to the MFMA's 16 rows is free), in bf16 the LDS transpose read does it.
//
// Neighbouring lanes of the K operand are different keys, a row apart in memory: loaded like that,
// every lane's 16 bytes are an access of their own to the vector cache, and the loads bound the
// kernel.  So K, and V in bf16, are loaded as they lie in memory, 1 KB of consecutive rows per
// instruction, and turned in a wavefront-private piece of LDS (no barrier), K chunks and V segments
// XOR-swizzled with the row (a round of 16 layers with D = 64: 339 -> 299 us; 8 layers in fp32:
// 224 -> 202).  The next tile's loads are issued as soon as the registers of the current one have gone to
// LDS.
//
// Latency: lengths -> page table -> first keys would be three dependent trips.  The table entries of a wavefront's tiles
// sit in one vector register (lane = tile and page, one trip for 32, fp32: 64, tiles) and are requested with the
// lengths, for the tiles the wavefront has if keys are not split over workgroups or the sequence fills its table;
// otherwise they are requested again.  Q and the ancestor masks follow and are not waited for.  With the pieces of the
// merge through LDS read all at once: rounds of 16 layers with D = 64 288 -> 272 us, 8 layers in fp32 191 -> 188,
// one small layer 18.1 -> 17.5.
#include <algorithm>
#include <type_traits>

#include "attn_direct.h"

namespace graft {

constexpr int PARTS_PAGES_128 = 48, PARTS_PAGES_128_RG1 = 30, PARTS_STEPS_128 = 4;              // (at plan_direct)
// Rows of a row block: 32 where a wavefront has that many and the products come in that size without a loss
constexpr int row_block_rows(bool bf16, int D, int mb) { return bf16 && D == 64 && mb >= 2 ? 32 : 16; }

// A lane's scores of one row block: 4 T values, value v = t[v / 4][v % 4].
template <int T> struct ScoreTiles {
    static constexpr int N = 4 * T;
    floatx4 t[T];
    __device__ __forceinline__ float get(int v) const { return t[v >> 2][v & 3]; }
    __device__ __forceinline__ void set(int v, float x) { t[v >> 2][v & 3] = x; }
};

constexpr bool shares_queries(bool f32, int D) { return f32 && D == 128; }

// Per storage type, head size and rows of a row block (RB): tile shape, LDS layout, the two products.
template <typename T, int D, int RB> struct DirectOps;

// K of a tile on its way from memory to LDS: 1 KB of consecutive rows per instruction.
template <int ROW, int TK> struct StagedKeys {
    static constexpr int N = TK * ROW / 1024, RPI = 1024 / ROW, CPR = ROW / 16;
    uintx4 r[N];
    static constexpr int page(int j) { return j * RPI / GRAFT_PAGE_SIZE; }
    static constexpr int row0(int j) { return j * RPI % GRAFT_PAGE_SIZE; }
    // row r of K to LDS, its 16-byte chunks in the order chunk ^ (r & 7)
    __device__ __forceinline__ void stage(unsigned char* Ks, int lane) const {
        const int lrow = lane / CPR, chunk = lane % CPR;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int row = j * RPI + lrow;
            *reinterpret_cast<uintx4*>(Ks + row * ROW + ((chunk ^ (row & 7)) * 16)) = r[j];
        }
    }
};

template <int D> struct DirectOps<float, D, 16> {
    static constexpr int TK = 16;               // keys per tile
    using Acc = floatx4;
    using Scores = ScoreTiles<1>;
    static constexpr int NO = D / 16, NP = D / 16;                // accumulators per row block, pieces of four dims
    static constexpr int key(int v) { return v; }                 // key of value v, apart from 4 (lane / RB)
    static constexpr int value_of(int key) { return key & 3; }    // and back: value, lane group
    static constexpr int group_of(int key) { return key >> 2 & 3; }
    static constexpr int ROW = D * 4;           // bytes
    static constexpr bool SUM_MFMA = false;
    static constexpr bool ALONE = true;         // values of any size: those of unseen slots do not reach a row even if they are not finite
    struct Q { floatx4 v[D / 16]; };
    static __device__ __forceinline__ void load_q(Q& q, const float* row, int lg) {
#pragma unroll
        for (int s = 0; s < D / 16; ++s) q.v[s] = *reinterpret_cast<const floatx4*>(row + 16 * s + 4 * lg);
    }
    // the same from LDS, where the chunks of row r are in the order chunk ^ (r & 7)
    static __device__ __forceinline__ void read_q(Q& q, const unsigned char* Qs, int row, int lg) {
#pragma unroll
        for (int s = 0; s < D / 16; ++s) q.v[s] = *reinterpret_cast<const floatx4*>(Qs + row * ROW + (((4 * s + lg) ^ (row & 7)) * 16));
    }
    template <int MB>
    static __device__ __forceinline__ void scores(const unsigned char* Ks, const Q (&q)[MB], Scores (&s)[MB], int l16, int lg) {
        const unsigned char* row = Ks + l16 * ROW;
        const int x = ((lg ^ l16) & 3) * 16 + (l16 & 4) * 16;      // chunk (4 d + lg) ^ (l16 & 7): bits 0-1 and, for even d, bit 2
#pragma unroll
        for (int d = 0; d < D / 16; ++d) {
            const floatx4 k = *reinterpret_cast<const floatx4*>(row + ((x ^ ((d & 1) * 64)) + (d >> 1) * 128));
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int rb = 0; rb < MB; ++rb)
                    s[rb].t[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[j], q[rb].v[d][j], d == 0 && j == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : s[rb].t[0], 0, 0, 0);
        }
    }
    static constexpr bool V_STAGED = false;     // values come in operand layout already: 256 bytes of a row per 16 lanes
    struct V { floatx4 r[4][D / 64]; };         // key 4 lg + i, dims 64 h + 4 l16 ..
    static __device__ __forceinline__ unsigned v_lane(int lane) { return 16 * (lane & 15); }
    static __device__ __forceinline__ int v_row(int lane, int j) { return 4 * (lane >> 4) + j; }
    static constexpr int NV = 4;                // row groups of a tile's values, page of each, its first row in the page
    static constexpr int v_page(int) { return 0; }
    static constexpr int v_row0(int j) { return j; }
    static __device__ __forceinline__ void load_v(V& t, int j, const char* base, unsigned off) {
#pragma unroll
        for (int h = 0; h < D / 64; ++h) t.r[j][h] = *reinterpret_cast<const floatx4*>(base + off + 256 * h);
    }
    template <int MB>
    static __device__ __forceinline__ void accumulate(const V& t, const unsigned char*, const Scores (&p)[MB], floatx4 (&o)[MB][NO],
                                                      floatx4 (&)[MB], int, int) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < D / 64; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int rb = 0; rb < MB; ++rb)
                        o[rb][4 * h + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.r[i][h][j], p[rb].t[0][i], o[rb][4 * h + j], 0, 0, 0);
    }
    // keys of the tile with an infinite or NaN value among this lane's, as bits
    static __device__ __forceinline__ unsigned nonfinite_keys(const V& t, int lane) {
        unsigned keys = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bool bad = false;
#pragma unroll
            for (int h = 0; h < D / 64; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i) bad = bad || !__builtin_isfinite(t.r[j][h][i]);
            keys |= bad ? 1u << j : 0u;
        }
        return keys << (4 * (lane >> 4));
    }
    static __device__ __forceinline__ void clear_key(V& t, unsigned char*, int key, int lane) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (4 * (lane >> 4) + j == key)
#pragma unroll
                for (int h = 0; h < D / 64; ++h) t.r[j][h] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    static __device__ __forceinline__ floatx4 load_dims(const char* p) { return *reinterpret_cast<const floatx4*>(p); }
    static __device__ __forceinline__ void add_piece(floatx4 (&o)[NO], int u, const floatx4& x) {
        const int h = u >> 2, i = u & 3;
#pragma unroll
        for (int j = 0; j < 4; ++j) o[4 * h + j][i] += x[j];
    }
    // the four consecutive dims starting at dim(u, lg), u < D/16
    static __device__ __forceinline__ int dim(int u, int lg) { return 64 * (u >> 2) + 16 * lg + 4 * (u & 3); }
    static __device__ __forceinline__ floatx4 piece(const floatx4 (&o)[NO], int u) {
        const int h = u >> 2, i = u & 3;
        return floatx4{o[4 * h][i], o[4 * h + 1][i], o[4 * h + 2][i], o[4 * h + 3][i]};
    }
};

// bf16: what does not depend on the rows of a block.
template <int D> struct DirectOpsBf16 {
    static constexpr int TK = 32;
    static constexpr int ROW = D * 2;
    static constexpr int P_PARTS = D == 64 ? 3 : 1;     // bf16 numbers that make up a probability (D = 128: rounded to one)
    static constexpr bool SUM_MFMA = P_PARTS == 1;      // row sums of the rounded probabilities, through the matrix cores
    static constexpr bool ALONE = D == 64;      // (D = 128 asks for finite, ordinary values, as the path this stands in for does)
    static constexpr int SEG = ROW / 32 - 1;    // V rows: 32-byte segment ^ (row & SEG)
    static constexpr bool V_STAGED = true;
    static constexpr int NV = TK * ROW / 1024, RPI = 1024 / ROW;       // instructions, rows per instruction
    struct V { uintx4 r[NV]; };
    static __device__ __forceinline__ unsigned v_lane(int lane) { return 16 * (lane % (ROW / 16)); }
    static __device__ __forceinline__ int v_row(int lane, int j) { return v_row0(j) + lane / (ROW / 16); }
    static constexpr int v_page(int j) { return j * RPI / GRAFT_PAGE_SIZE; }
    static constexpr int v_row0(int j) { return j * RPI % GRAFT_PAGE_SIZE; }
    static __device__ __forceinline__ void load_v(V& t, int j, const char* base, unsigned off) {
        t.r[j] = *reinterpret_cast<const uintx4*>(base + off);
    }
    // row r of V to LDS, its 32-byte segments in the order segment ^ (r & SEG)
    static __device__ __forceinline__ void stage_v(const V& t, unsigned char* Vs, int lane) {
        const int lrow = lane / (ROW / 16), chunk = lane % (ROW / 16);
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int row = j * RPI + lrow;
            *reinterpret_cast<uintx4*>(Vs + row * ROW + ((chunk ^ ((row & SEG) << 1)) * 16)) = t.r[j];
        }
    }
    static __device__ __forceinline__ unsigned nonfinite_keys(const V& t, int lane) {
        unsigned keys = 0;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            bool bad = false;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned x = t.r[j][i];
                bad = bad || (x & 0x7f80u) == 0x7f80u || (x & 0x7f800000u) == 0x7f800000u;
            }
            keys |= bad ? 1u << (j * RPI) : 0u;
        }
        return keys << (lane / (ROW / 16));
    }
    static __device__ __forceinline__ void clear_key(V&, unsigned char* Vs, int key, int lane) {
        if (lane < ROW / 16) *reinterpret_cast<uintx4*>(Vs + key * ROW + 16 * lane) = uintx4{0u, 0u, 0u, 0u};
    }
    static __device__ __forceinline__ floatx4 load_dims(const char* p) {
        const uintx2 x = *reinterpret_cast<const uintx2*>(p);
        return floatx4{__uint_as_float(x[0] << 16), __uint_as_float(x[0] & 0xffff0000u), __uint_as_float(x[1] << 16),
                       __uint_as_float(x[1] & 0xffff0000u)};
    }
    // What is left of a lane's probabilities and the next part of eight of them.  D = 64: p = part 0 + part 1 + part 2, each
    // the leading 8 bits of what the ones before it leave.  Both differences are exact, so no bit of p is lost: its products
    // with the bf16 values are those of fp32.  A part's MFMAs run while the next one is split off (four sequences of 2048
    // keys, 32 heads on 8: 15.5 us; 16.9 with all parts split off first and the row sums from the matrix cores, 14.8 with two
    // parts, 17 bits of p).
    template <class S> static __device__ __forceinline__ bf16x8 take_part(S& left, int v0) {
        uintx4 part;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float p0 = left.get(v0 + 2 * j), p1 = left.get(v0 + 2 * j + 1);
            if constexpr (P_PARTS == 1) {
                part[j] = pack_bf16(p0, p1);
            } else {
                const unsigned b0 = __float_as_uint(p0), b1 = __float_as_uint(p1);
                part[j] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
                left.set(v0 + 2 * j, p0 - __uint_as_float(b0 & 0xffff0000u));
                left.set(v0 + 2 * j + 1, p1 - __uint_as_float(b1 & 0xffff0000u));
            }
        }
        return __builtin_bit_cast(bf16x8, part);
    }
};

// bf16, 16 rows to a block: 16x16x32 MFMAs
template <int D> struct DirectOps<__bf16, D, 16> : DirectOpsBf16<D> {
    using Base = DirectOpsBf16<D>;
    using typename Base::V;
    using Base::ROW, Base::P_PARTS, Base::SUM_MFMA, Base::SEG;
    using Acc = floatx4;
    using Scores = ScoreTiles<2>;
    static constexpr int NO = D / 16, NP = D / 16;
    static constexpr int key(int v) { return 16 * (v >> 2) + (v & 3); }
    static constexpr int value_of(int key) { return (key >> 4) * 4 + (key & 3); }
    static constexpr int group_of(int key) { return key >> 2 & 3; }
    struct Q { bf16x8 v[D / 32]; };
    static __device__ __forceinline__ void load_q(Q& q, const __bf16* row, int lg) {
#pragma unroll
        for (int s = 0; s < D / 32; ++s) q.v[s] = *reinterpret_cast<const bf16x8*>(row + 32 * s + 8 * lg);
    }
    template <int MB>
    static __device__ __forceinline__ void scores(const unsigned char* Ks, const Q (&q)[MB], Scores (&s)[MB], int l16, int lg) {
        const unsigned char* row = Ks + l16 * ROW;
        const int x = ((lg ^ l16) & 3) * 16 + (l16 & 4) * 16;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int d = 0; d < D / 32; ++d) {
                const bf16x8 k = *reinterpret_cast<const bf16x8*>(row + ((x ^ ((d & 1) * 64)) + (d >> 1) * 128 + c * 16 * ROW));
#pragma unroll
                for (int rb = 0; rb < MB; ++rb)
                    s[rb].t[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k, q[rb].v[d], d == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : s[rb].t[c], 0, 0, 0);
            }
    }
    template <int MB>
    static __device__ __forceinline__ void accumulate(const V&, const unsigned char* Vs, const Scores (&p)[MB], floatx4 (&o)[MB][NO],
                                                      floatx4 (&sum)[MB], int l16, int lg) {
        // rows 16 c + 4 lg + (l16 >> 2): the transpose read turns 4 keys x 16 dims into "lane = dim, 4 keys"
        const int row0 = 4 * lg + (l16 >> 2);
        const unsigned base = lds_offset(Vs) + row0 * ROW + ((row0 & SEG) << 5) + 8 * (l16 & 3);
        bf16x8 a[NO];
#pragma unroll
        for (int e = 0; e < NO; ++e)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const short4_t r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (short4_t __attribute__((address_space(3)))*)(static_cast<size_t>((base ^ (e << 5)) + c * 16 * ROW)));
                const bf16x4 r4 = __builtin_bit_cast(bf16x4, r);
                a[e][4 * c] = r4[0];
                a[e][4 * c + 1] = r4[1];
                a[e][4 * c + 2] = r4[2];
                a[e][4 * c + 3] = r4[3];
            }
        Scores left[MB];
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) left[rb] = p[rb];
#pragma unroll
        for (int t = 0; t < P_PARTS; ++t)
#pragma unroll
            for (int rb = 0; rb < MB; ++rb) {
                const bf16x8 pp = Base::take_part(left[rb], 0);
#pragma unroll
                for (int e = 0; e < NO; ++e) o[rb][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[e], pp, o[rb][e], 0, 0, 0);
                if constexpr (SUM_MFMA) {
                    const bf16x8 ones = __builtin_bit_cast(bf16x8, uintx4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
                    sum[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pp, sum[rb], 0, 0, 0);
                }
            }
    }
    static __device__ __forceinline__ void add_piece(floatx4 (&o)[NO], int u, const floatx4& x) { o[u] += x; }
    static __device__ __forceinline__ int dim(int u, int lg) { return 16 * u + 4 * lg; }
    static __device__ __forceinline__ floatx4 piece(const floatx4 (&o)[NO], int u) { return o[u]; }
};

// bf16, 32 rows to a block: 32x32x16 MFMAs.  The kernel is bound by what a SIMD issues: a vector instruction takes 4 cycles, an
// exp2 8 and an MFMA of either size 8 of the same slots (measured with two and three wavefronts a SIMD; what is left of the
// MFMA's 16 or 32 cycles is free for others), so the larger ones cost half.  Four sequences of 2048 keys, 32 heads on 8: 15.3
// -> 14.0 us a layer; 16 sequences of 1024: 25.0 -> 23.0.  A third wavefront per SIMD (12 a workgroup) gains nothing.
// A: lane = key or dim (lane & 31), the 8 contraction indices of group lane / 32; B: lane = row; a result's value v is row
// (key or dim) 8 (v / 4) + 4 (lane / 32) + v % 4, so values 8 kk .. 8 kk + 7 are the second product's B operand for the
// 16 keys from 16 kk on, in the order in which the transpose read brings those of A.
template <int D> struct DirectOps<__bf16, D, 32> : DirectOpsBf16<D> {
    using Base = DirectOpsBf16<D>;
    using typename Base::V;
    using Base::ROW, Base::P_PARTS, Base::SEG;
    static_assert(!Base::SUM_MFMA && SEG == 3, "head size 64");
    using Acc = floatx16;
    struct Scores {
        static constexpr int N = 16;
        floatx16 t;
        __device__ __forceinline__ float get(int v) const { return t[v]; }
        __device__ __forceinline__ void set(int v, float x) { t[v] = x; }
    };
    static constexpr int NO = D / 32, NP = D / 8;
    static constexpr int key(int v) { return 8 * (v >> 2) + (v & 3); }
    static constexpr int value_of(int key) { return (key >> 3) * 4 + (key & 3); }
    static constexpr int group_of(int key) { return key >> 2 & 1; }
    struct Q { bf16x8 v[D / 16]; };
    static __device__ __forceinline__ void load_q(Q& q, const __bf16* row, int half) {
#pragma unroll
        for (int s = 0; s < D / 16; ++s) q.v[s] = *reinterpret_cast<const bf16x8*>(row + 16 * s + 8 * half);
    }
    template <int NB>
    static __device__ __forceinline__ void scores(const unsigned char* Ks, const Q (&q)[NB], Scores (&s)[NB], int l32, int half) {
        const unsigned char* row = Ks + l32 * ROW;
        const int x = ((half ^ l32) & 7) * 16;                    // chunk (2 d + half) ^ (l32 & 7)
#pragma unroll
        for (int d = 0; d < D / 16; ++d) {
            const bf16x8 k = *reinterpret_cast<const bf16x8*>(row + (x ^ (d * 32)));
#pragma unroll
            for (int rb = 0; rb < NB; ++rb) s[rb].t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, q[rb].v[d], d == 0 ? floatx16{} : s[rb].t, 0, 0, 0);
        }
    }
    template <int NB>
    static __device__ __forceinline__ void accumulate(const V&, const unsigned char* Vs, const Scores (&p)[NB], floatx16 (&o)[NB][NO],
                                                      floatx4 (&)[NB], int l32, int half) {
        // keys 16 kk + 8 c + 4 half + .., dims 32 e + l32: a 16-lane group of the transpose read has 4 keys and 16 dims
        const int l16 = l32 & 15, row0 = 4 * half + (l16 >> 2);
        const unsigned base = lds_offset(Vs) + row0 * ROW + (((l32 >> 4) ^ (row0 & SEG)) << 5) + 8 * (l16 & 3);
        bf16x8 a[NO][2];
#pragma unroll
        for (int e = 0; e < NO; ++e)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const short4_t r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (short4_t __attribute__((address_space(3)))*)(static_cast<size_t>((base ^ (e << 6)) + (16 * kk + 8 * c) * ROW)));
                    const bf16x4 r4 = __builtin_bit_cast(bf16x4, r);
                    a[e][kk][4 * c] = r4[0];
                    a[e][kk][4 * c + 1] = r4[1];
                    a[e][kk][4 * c + 2] = r4[2];
                    a[e][kk][4 * c + 3] = r4[3];
                }
        Scores left[NB];
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) left[rb] = p[rb];
#pragma unroll
        for (int t = 0; t < P_PARTS; ++t)
#pragma unroll
            for (int rb = 0; rb < NB; ++rb)
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    const bf16x8 pp = Base::take_part(left[rb], 8 * kk);
#pragma unroll
                    for (int e = 0; e < NO; ++e) o[rb][e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[e][kk], pp, o[rb][e], 0, 0, 0);
                }
    }
    static __device__ __forceinline__ void add_piece(floatx16 (&o)[NO], int u, const floatx4& x) {
#pragma unroll
        for (int i = 0; i < 4; ++i) o[u >> 2][4 * (u & 3) + i] += x[i];
    }
    static __device__ __forceinline__ int dim(int u, int half) { return 8 * u + 4 * half; }
    static __device__ __forceinline__ floatx4 piece(const floatx16 (&o)[NO], int u) {
        const int at = 4 * (u & 3);
        return floatx4{o[u >> 2][at], o[u >> 2][at + 1], o[u >> 2][at + 2], o[u >> 2][at + 3]};
    }
};

// p.R_pad = rows covered by the row tiles; rg (row groups) and the rest of the shape as below.  One row block
// with D = 64 leaves room for a second workgroup on the compute unit.
template <typename T, int D, int MB>
__global__ __launch_bounds__(DR_THREADS, MB * D == 64 ? 4 : 2) void tree_attn_direct_kernel(GRAFT_ATTN_ARGS) {
    constexpr int RB = row_block_rows(std::is_same_v<T, __bf16>, D, MB), NB = MB * 16 / RB;       // rows of a row block, row blocks
    using Ops = DirectOps<T, D, RB>;
    constexpr int TK = Ops::TK, NO = Ops::NO, NP = Ops::NP, NS = Ops::Scores::N, ROW = Ops::ROW;
    using Keys = StagedKeys<ROW, TK>;
    using Values = typename Ops::V;
    constexpr int STAGE = TK * ROW * (Ops::V_STAGED ? 2 : 1);   // a wavefront's piece of LDS: K, then V
    constexpr int PITCH = D + 4;                // LDS row pitch of the merge: 16 rows at consecutive 16-byte slots
    // fp32 with D = 128: the wavefronts of a row group request a share of its queries each and exchange them through LDS.  All
    // of them asking for all 8 KB kept the compute unit's address path busy for a microsecond in front of the first keys
    // (21.4 -> 20.9 us with 2K keys); with less to ask for, the barrier costs as much or more (D = 64: bf16 14.0 -> 14.4, fp32
    // 11.3 -> 11.6).  One key group has nothing to share.
    constexpr bool SHARE_Q = shares_queries(std::is_same_v<T, float>, D);
    constexpr bool MASK_HELD = MB * D < 256 && !SHARE_Q;          // the rows' ancestor masks in registers, else in LDS
    // the wavefronts' pieces (and the queries that are shared); after the loop, with more than one key group,
    // [wave][16 MB][PITCH] partial rows and (m, l) [wave][16 MB].  In front of it the ancestor masks, if they are held here.
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    unsigned char* const pieces = lds + (MASK_HELD ? 0 : DR_MASK_BYTES);
    float* const merge_lds = reinterpret_cast<float*>(pieces);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane % RB, lg = lane / RB;                     // row in a block, group of lanes
    const int rg = row_groups, kg = key_groups;
    const int kgi = div31(wave, row_groups_magic), rgi = wave - kgi * rg;
    const WorkItem item = xcd_work_item(n_units, n_row_tiles, row_tiles_magic);
    const bool padding = item.unit < 0;          // of the grid (whole workgroup): it leaves behind the first requests, which
                                                 // a branch in front of them would delay
    const int rt = item.row_tile, unit = padding ? 0 : item.unit;             // unit over B * Hkv * n_splits
    const int bg = div31(unit, splits_magic), split = unit - bg * n_splits;
    const int b = div24(bg, n_kv_heads), g = bg - b * n_kv_heads;

    const int b_lane = per_lane(b);              // (requested here, waited for behind the requests below)
    const int n_lane = n_nodes[b_lane], P_lane = prefix_len[b_lane];
    await_setup_args(p);
    if (padding) return;
    constexpr int PAGES = TK / GRAFT_PAGE_SIZE, TPR = 64 / PAGES;              // pages per tile, tiles per table register
    // The page table is requested before the lengths are known, for the tiles this wavefront has if the sequence fills
    // its table (with keys that are not split over workgroups: whatever its length).  Lane = ordinal of the tile, page.
    const int32_t* table = p.block_table + static_cast<size_t>(b) * p.max_pages;
    const int per_full = div31((p.max_pages + PAGES - 1) / PAGES + n_splits - 1, splits_magic);
    int tb = 0;
    {
        const int pg = (split * per_full + kgi + kg * (lane / PAGES)) * PAGES + lane % PAGES;
        tb = table[pg < p.max_pages ? pg : p.max_pages - 1];
    }
    const int r_base = (rt * rg + rgi) * (16 * MB);
    const auto query = [&](int r) __attribute__((always_inline)) {             // rows past R read row 0
        const int rc = r < p.R ? r : 0, i = (rc * p.g_magic) >> 16;
        return static_cast<const T*>(p.q) + ((static_cast<size_t>(b) * p.K_max + i) * p.Hq + (g * p.G + (rc - i * p.G))) * D;
    };
    constexpr int QN = SHARE_Q ? 16 * MB * ROW / 1024 : 2, QR = 1024 / ROW, CPR = ROW / 16;      // 1 KB pieces, rows of one, chunks of a row
    uintx4 q_share[QN / 2];
    typename Ops::Q q[NB];
    uintx4 mw[NB];                              // ancestor mask of the row's node
    int node[NB];
    if (SHARE_Q && kg > 1) {
#pragma unroll
        for (int u = 0; u < QN / 2; ++u) {
            const int j = kgi + u * kg;
            if (j < QN) q_share[u] = reinterpret_cast<const uintx4*>(query(r_base + j * QR + lane / CPR))[lane % CPR];
        }
    } else {
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) Ops::load_q(q[rb], query(r_base + rb * RB + lr), lg);
    }
#pragma unroll
    for (int rb = 0; rb < NB; ++rb) {
        const int r = r_base + rb * RB + lr;
        node[rb] = ((r < p.R ? r : 0) * p.g_magic) >> 16;
        if constexpr (MASK_HELD)
            mw[rb] = *reinterpret_cast<const uintx4*>(p.mask + (static_cast<size_t>(b) * p.K_max + node[rb]) * GRAFT_MASK_WORDS);
    }

    unsigned mask_word = 0;
    if constexpr (!MASK_HELD) {
        static_assert(GRAFT_MAX_NODES * 4 <= DR_THREADS, "one mask word per thread");
        if (tid < p.K_max * 4) mask_word = reinterpret_cast<const unsigned*>(p.mask + static_cast<size_t>(b) * p.K_max * GRAFT_MASK_WORDS)[tid];
    }

    __builtin_amdgcn_sched_barrier(0);
    const int n_raw = __builtin_amdgcn_readfirstlane(n_lane), P_raw = __builtin_amdgcn_readfirstlane(P_lane);
    int n = n_raw;
    if (n < 1 || n > p.K_max) n = 0;
    const int cap = p.max_pages * GRAFT_PAGE_SIZE;
    int P = P_raw;
    P = P < 0 ? 0 : (P > cap ? cap : P);
    const int total = n ? ((P + n) < cap ? (P + n) : cap) : 0;
    const int n_tiles = (total + TK - 1) / TK;
    const int per_split = div31(n_tiles + n_splits - 1, splits_magic);
    const int tile0 = split * per_split;
    const int tile1 = (tile0 + per_split) < n_tiles ? (tile0 + per_split) : n_tiles;
    // this wavefront's tiles: tile0 + kgi, + kg, ...; none if all its rows belong to absent nodes
    const int first = tile0 + kgi;
    const bool rows_live = ((r_base * p.g_magic) >> 16) < n && r_base < p.R;
    const int count = (rows_live && first < tile1) ? div31(tile1 - first + kg - 1, key_groups_magic) : 0;

    float m[NB], l[NB];
    floatx4 lv[NB];                             // row sums where the matrix cores take them (every entry the row's sum)
    typename Ops::Acc o[NB][NO];
    auto clear_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) {
            m[rb] = -INFINITY;
            l[rb] = 0.f;
            lv[rb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < NO; ++e) o[rb][e] = typename Ops::Acc{};
        }
    };
    clear_rows();

    const int last = total - 1, last_pg = last >> 4;
    const char* kc = static_cast<const char*>(p.k) + static_cast<int64_t>(g) * p.head_stride * sizeof(T);
    const char* vc = static_cast<const char*>(p.v) + static_cast<int64_t>(g) * p.head_stride * sizeof(T);
    const unsigned ts = static_cast<unsigned>(p.token_stride) * sizeof(T);   // bytes
    // Tiles in the order they are taken: the wavefront's last one first, so that the one tile of
    // the sequence that can reach past its end is only ever the first of a wavefront.  Loads
    // inside the loop then need no branch; with one, the compiler no longer knows how many
    // transfers are in flight and waits for most of what it has just requested.
    auto tile_at = [&](int it) __attribute__((always_inline)) { return first + kg * (it == 0 ? count - 1 : it - 1); };
    // (entries of the tiles it, it + 1, ...)
    auto load_table = [&](int it) __attribute__((always_inline)) {
        const int pg = tile_at(it + lane / PAGES) * PAGES + lane % PAGES;
        tb = table[pg < last_pg ? pg : last_pg];
    };
    // what was requested in front of the lengths serves if all tiles are in it and it began with the right one
    const bool in_order = count <= TPR && (n_splits == 1 || per_split == per_full);
    if (in_order) {
        if constexpr (PAGES > 1) {                                // a page past the last one repeats it
            const int tile = tile_at(0), over = last_pg - tile * PAGES;
            const int at = (count - 1) * PAGES + (over < PAGES - 1 ? over : PAGES - 1);
            const int entry = __builtin_amdgcn_readlane(tb, at & 63);
            tb = lane > at ? entry : tb;
        }
    } else if (count > 0) {
        load_table(0);
        asm volatile("" : "+v"(tb));                              // (waited for here: behind the join it would be for everything requested)
    }
    auto table_slot = [&](int it) __attribute__((always_inline)) {
        return in_order ? (it == 0 ? count - 1 : it - 1) & (TPR - 1) : it & (TPR - 1);
    };
    // (the wavefront-uniform part of an address is scalar, the lane's part loop-invariant)
    auto page_base = [&](int it, int c) __attribute__((always_inline)) {
        return static_cast<int64_t>(__builtin_amdgcn_readlane(tb, table_slot(it) * PAGES + c)) * p.page_stride * static_cast<int64_t>(sizeof(T));
    };
    const unsigned k_lane = 16 * (lane % Keys::CPR), k_off = lane / Keys::CPR * ts + k_lane;
    const unsigned v_lane = Ops::v_lane(lane), v_off = (Ops::v_row(lane, 0) - Ops::v_row0(0)) * ts + v_lane;
    auto load_keys = [&](Keys& t, int it) __attribute__((always_inline)) {
        unsigned off = k_off;
        asm volatile("" : "+v"(off));                         // (kept apart from the scalar base: no 64-bit vector additions)
#pragma unroll
        for (int j = 0; j < Keys::N; ++j)
            t.r[j] = *reinterpret_cast<const uintx4*>(kc + page_base(it, Keys::page(j)) + static_cast<int64_t>(Keys::row0(j)) * ts + off);
    };
    auto load_values = [&](Values& t, int it) __attribute__((always_inline)) {
        unsigned off = v_off;
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int j = 0; j < Ops::NV; ++j)
            Ops::load_v(t, j, vc + page_base(it, Ops::v_page(j)) + static_cast<int64_t>(Ops::v_row0(j)) * ts, off);
    };
    // a tile that may reach past the end: keys past the last token read the last token again
    // (its probability there is zero)
    auto row_off = [&](int it, int page, int k) __attribute__((always_inline)) {
        const int t_page = tile_at(it) * TK + 16 * page;
        const int lim = last - (t_page < last ? t_page : (last & ~15));
        return static_cast<unsigned>(k < lim ? k : lim) * ts;
    };
    auto load_clamped = [&](Keys& kt, Values& vt, int it) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < Keys::N; ++j)
            kt.r[j] = *reinterpret_cast<const uintx4*>(kc + page_base(it, Keys::page(j)) +
                                                       (row_off(it, Keys::page(j), Keys::row0(j) + lane / Keys::CPR) + k_lane));
#pragma unroll
        for (int j = 0; j < Ops::NV; ++j)
            Ops::load_v(vt, j, vc + page_base(it, Ops::v_page(j)), row_off(it, Ops::v_page(j), Ops::v_row(lane, j)) + v_lane);
    };
    unsigned char* const Ks = pieces + wave * STAGE;
    unsigned char* const Vs = Ks + TK * ROW;
    const float sc = p.scale_log2e;
    Keys kt;
    Values vt;
    if (count > 0) load_clamped(kt, vt, 0);
    const uintx4* mask_lds = reinterpret_cast<const uintx4*>(lds);
    if constexpr (!MASK_HELD) {                                   // (behind the first keys' request)
        if (tid < p.K_max * 4) reinterpret_cast<unsigned*>(lds)[tid] = mask_word;
        unsigned char* const Qs = pieces + DR_WAVES * STAGE + rgi * (16 * MB * ROW);
        if (SHARE_Q && kg > 1) {
#pragma unroll
            for (int u = 0; u < QN / 2; ++u) {
                const int j = kgi + u * kg, row = j * QR + lane / CPR;
                if (j < QN) *reinterpret_cast<uintx4*>(Qs + row * ROW + (((lane % CPR) ^ (row & 7)) * 16)) = q_share[u];
            }
        }
        lds_only_barrier();
        if constexpr (SHARE_Q) {
            if (kg > 1) {
#pragma unroll
                for (int rb = 0; rb < NB; ++rb) Ops::read_q(q[rb], Qs, rb * RB + lr, lg);
            }
        }
    }
    // One tile: through LDS where it has to be turned, the next one requested behind it.
    auto step = [&](int it, auto more_, auto careful_) __attribute__((always_inline)) {
        constexpr bool more = decltype(more_)::value, careful = decltype(careful_)::value;
        kt.stage(Ks, lane);
        asm volatile("" ::: "memory");                        // (lanes read each other's rows: no read moves in front of a write.
                                                              // Behind the next loads instead, it costs fp32 2 %.)
        if constexpr (more) load_keys(kt, it + 1);
        const int t0 = tile_at(it) * TK;
        const bool masked = t0 + TK > P;
        typename Ops::Scores s[NB];
        Ops::template scores<NB>(Ks, q, s, lr, lg);
        unsigned odd = 0;                                     // keys with an infinite or NaN value
        if constexpr (careful) {
            odd = Ops::nonfinite_keys(vt, lane);
#pragma unroll
            for (int x = 32; x >= 1; x >>= 1) odd |= __shfl_xor(odd, x);
            odd = __builtin_amdgcn_readfirstlane(odd);
        }
        if constexpr (Ops::V_STAGED) {
            Ops::stage_v(vt, Vs, lane);
            if constexpr (more) load_values(vt, it + 1);
        }
        if (__builtin_expect(masked, 0)) {
#pragma unroll
            for (int rb = 0; rb < NB; ++rb) {
                const uintx4 words = MASK_HELD ? mw[rb] : mask_lds[node[rb]];
                const unsigned win = visible_window(t0 - P, total - P, [&](int k) {
                    return k == 0 ? words[0] : (k == 1 ? words[1] : (k == 2 ? words[2] : words[3]));
                }) >> (4 * lg);
#pragma unroll
                for (int v = 0; v < NS; ++v) s[rb].set(v, keep_visible(s[rb].get(v), win, Ops::key(v)));
            }
        }
        float mx[NB];
        bool raise = false;
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) {
            // (two maxima an instruction; a row with a NaN among its scores is NaN either way)
            float x = s[rb].get(0);
#pragma unroll
            for (int v = 1; v < NS; ++v) x = __builtin_elementwise_maximum(x, s[rb].get(v));
            mx[rb] = x * sc;
            raise = raise || mx[rb] > m[rb] + (careful ? 0.f : DR_LAZY_LOG2);
        }
        // (rare) a row without a reference, or one that outgrew it: raise it to the maximum seen
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {
#pragma unroll
            for (int rb = 0; rb < NB; ++rb) {
                const float mn = fmaxf(m[rb], row_max<RB>(mx[rb]));
                const float a = mn == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m[rb] - mn);
                m[rb] = mn;
                l[rb] *= a;
                if constexpr (Ops::SUM_MFMA) lv[rb] *= a;
#pragma unroll
                for (int e = 0; e < NO; ++e) o[rb][e] *= a;
            }
        }
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) {
            const float neg = m[rb] == -INFINITY ? 0.f : -m[rb];
            float sum = 0.f;
#pragma unroll
            for (int v = 0; v < NS; ++v) {
                s[rb].set(v, __builtin_amdgcn_exp2f(__builtin_fmaf(s[rb].get(v), sc, neg)));
                if constexpr (!Ops::SUM_MFMA) sum += s[rb].get(v);
            }
            l[rb] += sum;
        }
        // the values of such a key leave the product and are added to the rows that see it
        for (unsigned left = odd; careful && left != 0; left &= left - 1) {
            const int key = __builtin_ctz(left), page = key >> 4, at = Ops::value_of(key);
            Ops::clear_key(vt, Vs, key, lane);
            const char* vrow = vc + page_base(it, page) + row_off(it, page, key & 15);
#pragma unroll
            for (int rb = 0; rb < NB; ++rb) {
                float pk = s[rb].get(0);
#pragma unroll
                for (int v = 0; v < NS; ++v) pk = at == v ? s[rb].get(v) : pk;
                pk = __shfl(pk, RB * Ops::group_of(key) + lr);
#pragma unroll
                for (int u = 0; u < NP; ++u) {
                    if (pk != 0.f) Ops::add_piece(o[rb], u, Ops::load_dims(vrow + Ops::dim(u, lg) * sizeof(T)) * pk);
                    asm volatile("" ::: "memory");            // (one load at a time: registers are short here)
                }
            }
        }
        asm volatile("" ::: "memory");                        // (the transpose reads stay behind the writes above)
        Ops::template accumulate<NB>(vt, Vs, s, o, lv, lr, lg);
        if constexpr (more && !Ops::V_STAGED) load_values(vt, it + 1);
    };
    // chunks of the tiles that one table register covers
    for (int it = 0; it < count;) {
        const int end = it + TPR < count ? it + TPR : count;
        if (it > 0) {
            load_table(it);
            load_clamped(kt, vt, it);
        }
        for (; it + 1 < end; ++it) step(it, std::true_type{}, std::false_type{});
        step(it, std::false_type{}, std::false_type{});
        it = end;
    }
    // ALONE: an infinite or NaN value in a tree slot makes the product NaN in the rows that do not see the slot as
    // well (0 * inf), and values past 2^112 can overflow against a lazy reference.  Such a wavefront, if there
    // ever is one, takes its tiles once more, with the values of such keys kept out of the product and the exact
    // running maximum.  (The same looked for in every step: 2 % on two row blocks with D = 64.)
    if constexpr (Ops::ALONE) {
        bool odd = false;
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) {
            float t = 0.f;                                    // two sums per instruction, NaN is kept
#pragma unroll
            for (int e = 0; e < NO; ++e)
#pragma unroll
                for (int i = 0; i < 4 * NP / NO; ++i) t = __builtin_elementwise_maximum(t, __builtin_fabsf(o[rb][e][i]));
            odd = odd || (!(t < INFINITY) && node[rb] < n);   // (queries of absent nodes may be anything)
        }
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd) != 0, 0)) {
            clear_rows();
            for (int it = 0; it < count; ++it) {
                if (!in_order && it % TPR == 0) load_table(it);
                load_clamped(kt, vt, it);
                step(it, std::false_type{}, std::true_type{});
            }
        }
    }
#pragma unroll
    for (int rb = 0; rb < NB; ++rb) l[rb] = Ops::SUM_MFMA ? lv[rb][0] : row_sum<RB>(l[rb]);

    // ---- results: this workgroup's rows, merged over its key groups
    T* outp = static_cast<T*>(p.out);
    float* ws_o = reinterpret_cast<float*>(p.ws_o);
    const size_t part = ((static_cast<size_t>(b) * n_kv_heads + g) * n_splits + split) * p.R_pad;
    if (kg == 1) {
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) {
            const int r = r_base + rb * RB + lr;
            if (n_splits == 1) {
                const bool keep = r < p.R && node[rb] < n && l[rb] > 0.f;
                const float inv = keep ? 1.0f / l[rb] : 0.f;
                T* row = outp + ((static_cast<size_t>(b) * p.K_max + node[rb]) * p.Hq + g * p.G + (r - node[rb] * p.G)) * D;
                if (r < p.R) {
#pragma unroll
                    for (int u = 0; u < NP; ++u) {
                        floatx4 x = Ops::piece(o[rb], u) * inv;
                        if (!keep) x = floatx4{0.f, 0.f, 0.f, 0.f};
                        store4(row + Ops::dim(u, lg), x);
                    }
                }
            } else {
#pragma unroll
                for (int u = 0; u < NP; ++u) store4(ws_o + (part + r) * D + Ops::dim(u, lg), Ops::piece(o[rb], u));
                if (lg == 0) {
                    p.ws_ml[2 * (part + r)] = m[rb];
                    p.ws_ml[2 * (part + r) + 1] = l[rb];
                }
            }
        }
        return;
    }
    __syncthreads();                                              // no wavefront reads its piece any more
    float* ml_lds = merge_lds + DR_WAVES * 16 * MB * PITCH;
#pragma unroll
    for (int rb = 0; rb < NB; ++rb) {
        float* row = merge_lds + (wave * 16 * MB + rb * RB + lr) * PITCH;
#pragma unroll
        for (int u = 0; u < NP; ++u) store4(row + Ops::dim(u, lg), Ops::piece(o[rb], u));
        if (lg == 0) {
            ml_lds[2 * (wave * 16 * MB + rb * RB + lr)] = m[rb];
            ml_lds[2 * (wave * 16 * MB + rb * RB + lr) + 1] = l[rb];
        }
    }
    __syncthreads();
    const int rows = rg * 16 * MB;                                // of this workgroup
    const auto merge = [&](auto kg_) __attribute__((always_inline)) {
        merge_key_groups<T, D, decltype(kg_)::value>(p, merge_lds, ml_lds, rows, rt * rows, tid, b, g, n, n_splits, part);
    };
    if (kg == 8) merge(std::integral_constant<int, 8>{});
    else if (kg == 4) merge(std::integral_constant<int, 4>{});
    else merge(std::integral_constant<int, 2>{});
}

// Merge of the splits: one thread per four dims of a row, the splits' pieces requested U at a time, all of them in flight: buffer
// loads, zeros where there is no split (with a condition around each, a split was waited for before the next was requested).  8 layers of
// 2K keys in fp32 (6 splits) 165.9 -> 157.3 us.  R_magic: magic31(R), exact as a
// job is split only while it has at most 4 units a compute unit, of 512 rows at most (2^19 rows, R <= 2048).
template <typename T, int D, int U>
__global__ __launch_bounds__(256) void tree_attn_direct_merge_kernel(
    const unsigned short* ws_bits, const float* ws_ml, const int32_t* n_nodes, int32_t n_rows, int32_t R, uint32_t R_magic, int32_t R_pad,
    int32_t n_splits, int32_t n_kv_heads, AttnParams p) {
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int row = x / (D / 4) < n_rows ? x / (D / 4) : n_rows - 1, d4 = x % (D / 4);         // row over B * Hkv * R
    const int bg = div31(row, R_magic), r = row - bg * R;
    // from the (b, g) of the wavefront's first row on, of which it has at most 64 / (D / 4)
    const int bg0 = __builtin_amdgcn_readfirstlane(bg);
    const size_t row0 = static_cast<size_t>(bg0) * n_splits * R_pad;
    const unsigned bytes = 0x7fffffffu;
    const auto o_rows = merge_buffer(reinterpret_cast<const float*>(ws_bits) + row0 * D, bytes), ml_rows = merge_buffer(ws_ml + row0 * 2, bytes);
    const unsigned at = (bg - bg0) * n_splits * R_pad + r;
    float mm = -INFINITY, den = 0.f;
    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
    int n = 0, b = 0;
    for (int s0 = 0; s0 < n_splits; s0 += U) {
        float2 ml[U];
        floatx4 ov[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned i = s0 + u < n_splits ? (at + (s0 + u) * R_pad) * 8 : ~7u;
            ml[u] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(ml_rows, i, 0, 0));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned i = s0 + u < n_splits ? (at + (s0 + u) * R_pad) * (4 * D) + 16 * d4 : ~15u;
            ov[u] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(o_rows, i, 0, 0));
        }
        if (s0 == 0) {
            b = div24(bg, n_kv_heads);
            n = n_nodes[b];
            asm volatile("" : : "s"(p.out), "s"(p.K_max), "s"(p.Hq), "s"(p.G), "s"(p.g_magic));
        }
        __builtin_amdgcn_sched_barrier(0);
        float mx = mm;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + u >= n_splits) ml[u].x = -INFINITY;
            mx = fmaxf(mx, ml[u].x);
        }
        const float keep = mm == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mm - mx);
        den *= keep;
        acc *= keep;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float f = ml[u].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[u].x - mx);
            den += f * ml[u].y;
            acc += ov[u] * f;
        }
        mm = mx;
    }
    if (x / (D / 4) >= n_rows) return;
    const int g = bg - b * n_kv_heads;
    if (n < 1 || n > p.K_max) n = 0;
    const int i = (r * p.g_magic) >> 16;
    const bool keep = i < n && den > 0.f;
    const floatx4 y = keep ? acc * (1.0f / den) : floatx4{0.f, 0.f, 0.f, 0.f};
    store4(static_cast<T*>(p.out) + ((static_cast<size_t>(b) * p.K_max + i) * p.Hq + g * p.G + (r - i * p.G)) * D + 4 * d4, y);
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
static size_t direct_lds_bytes(int mb, int rg, int32_t D, int32_t dtype) {
    const bool share = shares_queries(dtype == GRAFT_F32, D);
    const size_t row = static_cast<size_t>(D) * (dtype == GRAFT_F32 ? 4 : 2);
    size_t loop = static_cast<size_t>(DR_WAVES) * (dtype == GRAFT_F32 ? 16 : 2 * 32) * row, merge = 0;
    if (rg < DR_WAVES) {
        if (share) loop += static_cast<size_t>(rg) * 16 * mb * row;
        merge = static_cast<size_t>(DR_WAVES) * 16 * mb * (D + 4 + 2) * sizeof(float);
    }
    return (loop > merge ? loop : merge) + (mb * D >= 256 || share ? DR_MASK_BYTES : 0);
}

// Launch shape: row blocks per wavefront, row groups per workgroup and splits that make the
// estimated time smallest.  One workgroup of eight wavefronts (two per SIMD) is resident per
// compute unit, so the job runs in ceil(workgroups / CUs) rounds of a fixed part plus a step per
// tile of a wavefront.  Cycles of a step (eight wavefronts, one tile each): fp32 4700 / 8200
// (D = 128, one / two row blocks) and 2650 (D = 64), against 4096 / 8192 and 2048 of MFMAs on a SIMD;
// bf16 2600 (D = 128) and, for D = 64, 1700 / 2750 / 4550 for one / two / four row blocks.  Measured with
// 256 workgroups, keys shared by 16 row tiles: 2130 / 3960, 1130, 1335 and 825 / 1270 / 2045 ns, the
// same at 2 to 2.3 GHz (the blocks of 32 rows took 2 to 4 % off the steps of 16-row blocks they replaced, 1300 / 2080, and
// the rest of their gain off the fixed part).  Set-up and the merge through LDS take 6500 + 2000 per row block and 64 dims
// (bf16 with D = 64, one / two / four row blocks: 4.0 / 4.2 / 7.3 us, launch included); the merge of splits is a launch of
// its own, 8000 + 600 per split and its traffic, 8 bytes per partial value at 3200 bytes per cycle.
DirectPlan plan_direct(int32_t B, int32_t K_max, int32_t Hq, int32_t Hkv, int32_t D, int32_t max_pages, int32_t dtype,
                       bool may_split) {
    DirectPlan best{};
    best.cost = -1.0;
    const int R = K_max * (Hq / Hkv), blocks = (R + 15) / 16;
    const int TK = dtype == GRAFT_F32 ? 16 : 32;
    const int64_t tiles = (static_cast<int64_t>(max_pages) * GRAFT_PAGE_SIZE + TK - 1) / TK;
    const int64_t cus = device_compute_units();
    const int mb_max = dtype == GRAFT_F32 ? (D == 128 ? 2 : 1) : (D == 128 ? 1 : 4);
    const double rows = static_cast<double>(B) * Hkv * R;
    const auto merge_cost = [&](int sp) { return sp > 1 ? 8000.0 + 600.0 * sp + sp * rows * D / 400.0 : 0.0; };
    const auto rounds_of = [&](int64_t workgroups) { return static_cast<double>((workgroups + cus - 1) / cus); };
    const auto plan_cost = [&](int mb, int64_t per, int64_t workgroups, int sp) {
        double c_step = D == 64 ? 2650.0 : (mb == 1 ? 4700.0 : 8200.0);
        if (dtype != GRAFT_F32 && D == 128) c_step = 2600.0;
        else if (dtype != GRAFT_F32) c_step = mb == 4 ? 4550.0 : (mb == 2 ? 2750.0 : 1700.0);
        const double c_fixed = 6500.0 + 2000.0 * mb * (D / 64);
        return rounds_of(workgroups) * (c_fixed + per * c_step) + merge_cost(sp);
    };
    for (int mb = 1; mb <= mb_max; mb *= 2) {
        for (int rg = 1; rg <= DR_WAVES; rg *= 2) {
            const int kg = DR_WAVES / rg;
            const int n_rt = (blocks + rg * mb - 1) / (rg * mb);
            if (rg > 1 && (rg / 2) * mb >= blocks) break;          // half the row groups would do
            const int64_t units = static_cast<int64_t>(B) * Hkv * n_rt;
            for (int sp = 1; sp <= (may_split ? DR_MAX_SPLITS : 1); ++sp) {
                const int64_t per = (tiles + static_cast<int64_t>(sp) * kg - 1) / (static_cast<int64_t>(sp) * kg);
                const double cost = plan_cost(mb, per, units * sp, sp);
                if (best.cost < 0.0 || cost < best.cost) best = {mb, rg, n_rt, sp, 0, 0, 0, cost, false};
                if (units * sp > 4 * cus || per <= 1) break;
            }
        }
    }
    // fp32 on the 16-bit matrix cores (tree_attn_parts.hip): 32 rows and eight key groups a workgroup, tiles of 32 keys.  A step is 5.05 us
    // with D = 128 and 2.95 with D = 64; one that not all wavefronts have takes its share, at least half (their SIMDs are their own).  At the
    // fp32 costs' 2133 a us that is 10800 and 6250, but those plans take longer than their costs by as much: 110 drawn shapes of 4 to 40
    // steps a compute unit take 0.828 of the time with fp32 products where the choice is made with 8150, 0.828 with 8800, 0.836 with 9500
    // and 0.849 with 10800; with D = 64 5300 (by 4750, 2 of 88 drawn shapes that take 1.10 and 1.11 times the time so).
    // D = 128 with short tables: us a call with fp32 MFMAs / with parts.  Of PARTS_STEPS_128 steps a compute unit or more, 10 x 564 tokens, 1936
    // rows, 74.2 / 52.0, 30 of 490 x 676 69.0 / 46.3, 56 of 283 x 645 76.5 / 57.2, 28 of 669 x 1176 150 / 94.  Of fewer, with one row group in the
    // fp32 plan: from PARTS_PAGES_128_RG1 pages on 24.2 / 16.1 (467 tokens, 1694 rows on 4 heads); of 26 pages 12.6 / 14.5 (410, 630 on 2) and
    // 13.7 / 15.4 (414, 896 on 4).  With several row groups they stay with fp32 MFMAs: tests/test_gpu_attn_direct.py holds the row groups (2, 4
    // and 8) of that kernel to such shapes, which costs speed there: 256 workgroups of 256 keys take 15.5 us so and 11.9 with parts.
    const int n_rt32 = (R + 31) / 32;
    const int64_t tiles32 = (static_cast<int64_t>(max_pages) + 1) / 2, units32 = static_cast<int64_t>(B) * Hkv * n_rt32;
    const bool parts_128 = max_pages >= PARTS_PAGES_128 || (best.rg == 1 && max_pages >= PARTS_PAGES_128_RG1) ||
                           units32 * tiles32 >= PARTS_STEPS_128 * DR_WAVES * cus;
    if (dtype == GRAFT_F32 && (D == 64 || parts_128)) {
        const double c_step = D == 64 ? 5300.0 : 8150.0, c_fixed = D == 64 ? 12000.0 : 14500.0;
        const double ahead = D == 64 || max_pages >= PARTS_PAGES_128 ? 1.0 : 0.95;      // (a step or two a compute unit: the costs are no better than that)
        const auto parts_cost = [&](int sp, int64_t of) {
            const int64_t per = (of + sp - 1) / sp, over = per % DR_WAVES;
            const double steps = static_cast<double>(per / DR_WAVES) + (over ? std::max(0.5, over / static_cast<double>(DR_WAVES)) : 0.0);
            return rounds_of(units32 * sp) * (c_fixed + steps * c_step) + merge_cost(sp);
        };
        const DirectPlan fp32 = best;
        for (int sp = 1; sp <= (may_split ? DR_MAX_SPLITS : 1); ++sp) {
            const double cost = parts_cost(sp, tiles32);
            if (cost < (best.parts ? 1.0 : ahead) * best.cost) best = {2, 1, n_rt32, sp, 0, 0, 0, cost, true};
            if (units32 * sp > 4 * cus || (tiles32 + sp - 1) / sp <= DR_WAVES / 2) break;
        }
        // Not split, a workgroup's fixed part (5.6 us with D = 64, 6.8 with 128) is what the other kernel's short steps are compared with, and a
        // table seldom is full: less than 9 per cent ahead here, it has to be ahead with half the keys too.  170 drawn shapes of 32 to 16384 tokens, time
        // over that with fp32 products with a full table / half the keys / an eighth: without this (and 4750 for the step with D = 64) 0.740 (largest
        // 1.11) / 0.804 (1.25) / 0.916 (1.71), with it 0.741 (1.02) / 0.799 (1.24) / 0.906
        // (1.42); 170 shapes that the line was not drawn by 0.741 (1.02) / 0.797 (1.18) / 0.902 (1.54).
        if (best.parts && best.n_splits == 1 && best.cost >= 0.91 * fp32.cost) {
            const int64_t each = static_cast<int64_t>(fp32.n_splits) * (DR_WAVES / fp32.rg), units = static_cast<int64_t>(B) * Hkv * fp32.n_row_tiles;
            const double half = plan_cost(fp32.mb, ((tiles + 1) / 2 + each - 1) / each, units * fp32.n_splits, fp32.n_splits);
            if (parts_cost(1, (tiles32 + 1) / 2) >= half) best = fp32;
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
static int32_t launch_rows(const DirectPlan& pl, const AttnParams& p, int32_t dtype, hipStream_t s) {
    return launch_pieces<T, D, tree_attn_direct_kernel<T, D, MB>>(pl, p, static_cast<unsigned>(direct_lds_bytes(MB, pl.rg, D, dtype)), s);
}
template <typename T, int D>
static int32_t launch_merge(int32_t rc, const DirectPlan& pl, const AttnParams& p, hipStream_t s) {
    if (rc != GRAFT_OK || pl.n_splits == 1) return rc;
    // (keys are split only while the chip is not full: one piece, few rows)
    const int64_t n_rows = static_cast<int64_t>(p.B) * p.Hkv * p.R;
    const auto merge = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((n_rows * (D / 4) + 255) / 256)), dim3(256), 0, s, p.ws_o, p.ws_ml, p.n_nodes,
                           static_cast<int32_t>(n_rows), p.R, magic31(static_cast<uint32_t>(p.R)), p.R_pad, p.n_splits, p.Hkv, p);
    };
    if (p.n_splits > 8) merge(tree_attn_direct_merge_kernel<T, D, 16>);
    else merge(tree_attn_direct_merge_kernel<T, D, 8>);
    return check_launch();
}

int32_t launch_direct(const DirectPlan& pl, AttnParams p, int32_t D, int32_t dtype, void* workspace, hipStream_t s) {
    p.n_splits = pl.n_splits;
    p.n_row_tiles = pl.n_row_tiles;
    p.R_pad = pl.r_pad;
    p.ws_o = static_cast<unsigned short*>(workspace);
    p.ws_ml = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + pl.ws_o_bytes);
    if (dtype == GRAFT_F32) {
        if (D == 64) return launch_merge<float, 64>(pl.parts ? launch_parts(pl, p, D, s) : launch_rows<float, 64, 1>(pl, p, dtype, s), pl, p, s);
        const int32_t rc = pl.parts ? launch_parts(pl, p, D, s) : (pl.mb == 1 ? launch_rows<float, 128, 1>(pl, p, dtype, s) : launch_rows<float, 128, 2>(pl, p, dtype, s));
        return launch_merge<float, 128>(rc, pl, p, s);
    }
    if (D == 128) return launch_merge<__bf16, 128>(launch_rows<__bf16, 128, 1>(pl, p, dtype, s), pl, p, s);
    const int32_t rc = pl.mb == 4 ? launch_rows<__bf16, 64, 4>(pl, p, dtype, s) : (pl.mb == 1 ? launch_rows<__bf16, 64, 1>(pl, p, dtype, s) : launch_rows<__bf16, 64, 2>(pl, p, dtype, s));
    return launch_merge<__bf16, 64>(rc, pl, p, s);
}

}  // namespace graft
