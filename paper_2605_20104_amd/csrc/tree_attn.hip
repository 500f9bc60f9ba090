// graft_tree_attn: tree-masked GQA attention over a paged KV cache.
//
// Two code paths.
//
// (1) bf16, D = 128, except where the keys are few: split-KV MFMA kernel + log-sum-exp combine.
//     All R = K_max * (Hq/Hkv) query rows of one KV head share every K/V element
//     that is streamed, so K and V are read from HBM once per head; the
//     arithmetic intensity is R flop per byte, which puts the tree-verify shapes
//     (R = 160..768) around the MFMA/HBM ridge of the chip.
//       grid  : one workgroup of 256 threads (4 wavefronts, one per SIMD, 512
//               registers each) per (row tile, split, KV head, sequence); the
//               host plan sizes it to about one workgroup per compute unit.
//       rows  : a wavefront owns 16*MB query rows (MB = 1, 2, 3 or 5 MFMA row blocks).  Its
//               O^T accumulators and the Q operand live in hand-placed AccVGPRs
//               and are only touched by inline-asm MFMAs inside the loop.
//       K/V   : 64-token stages (4 pages) go global -> LDS directly (no register
//               staging) into a ring of four buffers, two stages in flight, one
//               LDS-only barrier per stage; K rows are XOR-swizzled at 16 B and
//               V rows at 32 B so that the MFMA operand reads spread over all banks.
//       QK^T  : X^T = K * Q'^T - m with v_mfma_f32_16x16x32_bf16, where
//               Q' = bf16(Q * scale * log2 e) and the negated row reference m is
//               the accumulator input: the result is the argument of exp2.  Each
//               lane holds exponents of ONE query row (column l%16), and the
//               packed probabilities are already laid out as the B operand of
//               the second product (no LDS round trip).
//       PV    : O^T += V^T * P^T; the V^T operand (contraction over tokens, which
//               are strided in memory) comes from the gfx950 LDS transpose read
//               ds_read_b64_tr_b16: a 16-lane group turns a 4-token x 16-dim
//               block into "lane = dim, 4 tokens packed".  Row sums: one more
//               MFMA per row block with an all-ones A operand.
//       pipeline: over 32-token sub-tiles, MFMAs of one sub-tile interleaved slot
//               by slot with the exp2 / pack / max work of its neighbours; the
//               MFMA operands are read from LDS two or three groups ahead,
//               across the boundary between the two regions of a step.
//       mask  : only sub-tiles that reach past the prefix take the masked path
//               (ancestor bits from graft_build_tree_mask); the prefix is dense.
//       softmax: a row's reference is the maximum of the first sub-tile that gives
//               it a finite score and is kept while later exponents stay below
//               2^24; beyond that the wavefront switches to an exact online
//               softmax loop that rescales the accumulators.
//     With one split per (sequence, KV head) the rows are normalised and written as
//     bf16 straight from the accumulators.  Otherwise partials (reference, sum, and
//     O / sum as fp16 rows with a per-row scale) go to the workspace; a small combine
//     kernel merges the splits and writes bf16.
//
//     Long key ranges with many rows take tiles of 192, 256 or 384 rows in blocks of 32 instead:
//     tree_attn_wide.hip, with the same stages and workspace sizes; the plan and the merge are here.
//
// (2) fp32 storage, D = 64, and bf16 with D = 128 where the keys are few: tree_attn_direct.hip.
#include <cstring>

#include "attn_mfma.h"

namespace graft {

constexpr float AT_LAZY_LOG2 = 24.0f;  // a row keeps its reference while exponents stay below 2^24

// ---------------------------------------------------------------------------
// path (1): MFMA split-KV kernel
// ---------------------------------------------------------------------------

// ---- MFMA issue through inline assembly, accumulators in fixed AccVGPRs ----------------
// With 512 registers per lane available the register allocator rotates MFMA accumulators
// between register sets, parks them in AccVGPRs and copies them back for every vector ALU
// use.  Here the placement is part of the design and is done by hand:
//   O^T accumulators of row block rb, dim block db : a[32 rb + 4 db .. +3], accumulated in
//       place and never touched by the vector ALUs inside the fast loop;
//   Q^T operand of row block rb < QA, dim step ds   : a[32 MB + 16 rb + 4 ds .. +3];
//   row sums of row block rb < 4                     : a[48 MB + 4 rb .. +3] (a fifth row block's
//       are in VGPRs: 48 * 5 + 16 = 256 is the whole AccVGPR file);
//   score tiles, probabilities, K/V operands        : VGPRs chosen by the compiler.
// The compiler itself uses no AccVGPR in this kernel (VGPR-to-AccVGPR spilling is switched
// off in the build, and the kernel must compile without spills); the asm statement in
// reserve_acc_registers() lists the hand-managed ones as clobbered so that they are counted in
// the kernel's register allocation; it is repeated inside the loops so that the compiler never
// parks a value of its own in one of them across the MFMAs.  asm volatile statements keep
// their relative order, which also pins the MFMA sequence.
// Hazards handled by construction: no vector ALU, LDS or memory instruction touches an MFMA
// result within 16 instructions of the MFMA (the pipeline regions are far apart and explicit
// s_nop guards the other places), dependent MFMAs on one accumulator are at least two
// instructions apart, AccVGPR writes are followed by s_nop before an MFMA reads them, an MFMA
// that may have a vector ALU write of one of its VGPR sources right in front of it (the first
// of a pipeline region, all of the slow path) begins with s_nop 1, and constants used as MFMA
// sources are made opaque to the compiler.  The build checks the generated assembly for the
// source-write distance, for compiler use of the hand-managed registers and for spills.
template <int MB> constexpr int q_in_acc() { return MB; }   // row blocks with Q^T in AccVGPRs (all, for MB <= 5)
constexpr int L_IN_ACC = 4;                                  // row blocks with their row sums in AccVGPRs
template <int MB> constexpr int acc_used() { return 32 * MB + 16 * q_in_acc<MB>() + 4 * (MB < L_IN_ACC ? MB : L_IN_ACC); }
constexpr int o_reg(int rb, int db) { return 32 * rb + 4 * db; }
template <int MB> constexpr int q_reg(int rb, int ds) { return 32 * MB + 16 * rb + 4 * ds; }
template <int MB> constexpr int l_reg(int rb) { return 48 * MB + 4 * rb; }

template <int MB>
__device__ __forceinline__ void reserve_acc_registers() {
    asm volatile("" ::: GRAFT_ACC_BLOCK_0);
    if constexpr (acc_used<MB>() > 48) asm volatile("" ::: GRAFT_ACC_BLOCK_1);
    if constexpr (acc_used<MB>() > 96) asm volatile("" ::: GRAFT_ACC_BLOCK_2);
    if constexpr (acc_used<MB>() > 144) asm volatile("" ::: GRAFT_ACC_BLOCK_3);
    if constexpr (acc_used<MB>() > 192) asm volatile("" ::: GRAFT_ACC_BLOCK_4);
    if constexpr (acc_used<MB>() > 240) asm volatile("" ::: GRAFT_ACC_BLOCK_5);
}

// The compiler does not know that these asm statements are MFMAs, so it inserts none of the
// wait states an MFMA needs after a vector ALU write of one of its VGPR sources (2 for the
// A and B operands, 1 for C: measured on gfx950, a shorter distance makes the MFMA read the
// old register contents).  Two mechanisms cover this: GUARD = true puts s_nop 1 in front of
// the MFMA (used wherever the preceding instructions are the compiler's choice and the cost
// does not matter), and the build checks the generated assembly of this file and fails if
// any MFMA has a vector ALU write of one of its sources within the two preceding
// instructions.  Constants used as MFMA sources are made opaque to the compiler so that it
// cannot rematerialise them in front of the statement.
#define GRAFT_MFMA_GUARD "s_nop 1\n\t"
// exponent tile (VGPRs) = K operand (VGPRs) x Q'^T operand (fixed AccVGPRs) + C, where C is the
// tile being accumulated or, for the first dim step, the row's negated reference.
template <int QR, bool GUARD = false>
__device__ __forceinline__ void mfma_x_first(floatx4& d, const bf16x8& ka, const floatx4& c) {
    if constexpr (GUARD)
        asm volatile(GRAFT_MFMA_GUARD "v_mfma_f32_16x16x32_bf16 %0, %1, a[%2:%3], %4"
                     : "=&v"(d) : "v"(ka), "n"(QR), "n"(QR + 3), "v"(c));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, a[%2:%3], %4"
                     : "=&v"(d) : "v"(ka), "n"(QR), "n"(QR + 3), "v"(c));
}
template <int QR, bool GUARD = false>
__device__ __forceinline__ void mfma_x_next(floatx4& d, const bf16x8& ka) {
    if constexpr (GUARD)
        asm volatile(GRAFT_MFMA_GUARD "v_mfma_f32_16x16x32_bf16 %0, %1, a[%2:%3], %0"
                     : "+v"(d) : "v"(ka), "n"(QR), "n"(QR + 3));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, a[%2:%3], %0" : "+v"(d) : "v"(ka), "n"(QR), "n"(QR + 3));
}
// O^T tile (fixed AccVGPRs) += V^T operand (VGPRs) x P^T operand (VGPRs)
template <int OR, bool GUARD = false>
__device__ __forceinline__ void mfma_o(const bf16x8& va, const uintx4& pb) {
    if constexpr (GUARD)
        asm volatile(GRAFT_MFMA_GUARD "v_mfma_f32_16x16x32_bf16 a[%0:%1], %2, %3, a[%0:%1]"
                     : : "n"(OR), "n"(OR + 3), "v"(va), "v"(pb));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 a[%0:%1], %2, %3, a[%0:%1]"
                     : : "n"(OR), "n"(OR + 3), "v"(va), "v"(pb));
}
// row sums += ones x P^T operand: every element of the tile ends up holding the row's sum.
// In AccVGPRs a[LR .. LR+3], or (a fifth row block) in VGPRs.
template <int LR, bool GUARD = false>
__device__ __forceinline__ void mfma_rowsum_acc(const bf16x8& ones, const uintx4& pb) {
    if constexpr (GUARD)
        asm volatile(GRAFT_MFMA_GUARD "v_mfma_f32_16x16x32_bf16 a[%0:%1], %2, %3, a[%0:%1]" : : "n"(LR), "n"(LR + 3), "v"(ones), "v"(pb));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 a[%0:%1], %2, %3, a[%0:%1]" : : "n"(LR), "n"(LR + 3), "v"(ones), "v"(pb));
}
template <bool GUARD = false>
__device__ __forceinline__ void mfma_rowsum(floatx4& l, const bf16x8& ones, const uintx4& pb) {
    if constexpr (GUARD)
        asm volatile(GRAFT_MFMA_GUARD "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(l) : "v"(ones), "v"(pb));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(l) : "v"(ones), "v"(pb));
}
// What one wavefront keeps in VGPRs for its 16*MB query rows (O^T and Q'^T are in AccVGPRs).
// Exponents are in log2 units throughout: Q' = bf16(Q * scale * log2 e), so that the MFMA
// result q'.k - m_ref is directly the argument of exp2.
template <int MB>
struct WaveRows {
    floatx4 negm[MB];       // {-m_ref} x 4: accumulator input of the first QK^T step (0 while unset);
                            // m_ref is the reference max of the row in log2 units
    floatx4 lsum_v;         // row sums of a fifth row block (the others' are in AccVGPRs)
    float thr[MB];          // an exponent above this needs attention: -inf while the row has no reference
                            // yet, else the lazy bound
    float thr_min;          // the smallest of thr[]: one compare of the largest new exponent against it
                            // decides whether any row needs attention (the rows are then looked at one by one)
    __device__ __forceinline__ bool unset(int rb) const { return thr[rb] == -INFINITY; }
    __device__ __forceinline__ float m_ref(int rb) const { return unset(rb) ? -INFINITY : -negm[rb][0]; }
};

// LDS byte offsets of this lane's MFMA operands inside a 32-token sub-tile.
// K group g = (c, ds): rows 16c + l16, 16-byte chunk (4ds + lg) ^ l16.
__device__ __forceinline__ bf16x8 load_k_operand(const unsigned char* Ks, int g, int l16, int lg) {
    const int c = g >> 2, ds = g & 3;
    return *reinterpret_cast<const bf16x8*>(Ks + (16 * c + l16) * AT_ROW_BYTES + (((4 * ds + lg) ^ l16) * 16));
}
// V^T operand of dim block db through the LDS transpose read: a 16-lane group turns the
// 4-token x 16-dim block (tokens 16c + 4lg .. +3, dims 16db .. +15) into "lane = dim, 4 tokens".
// (half c = tokens 16c .. 16c + 15 of the sub-tile: one transpose read, elements 4c .. 4c + 3)
template <int C>
__device__ __forceinline__ void load_v_half(bf16x8& va, const unsigned char* Vs, int db, int l16, int lg) {
    // row 16C + 4lg + (l16 >> 2), 32-byte segment db ^ (row & 7): the segment is bits 5-7 of the
    // address, row & 7 does not depend on C, and sub-tiles start at multiples of 256 bytes, so
    // the address is the lane's base (which carries row & 7 in those bits) XOR db << 5, plus a
    // constant for C that fits the read's offset field: one vector instruction per dim block.
    const int row0 = 4 * lg + (l16 >> 2);
    const unsigned base = lds_address(Vs) + row0 * AT_ROW_BYTES + ((row0 & 7) << 5) + 8 * (l16 & 3);
    const short4_t r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (short4_t __attribute__((address_space(3)))*)(static_cast<size_t>((base ^ (db << 5)) + C * 16 * AT_ROW_BYTES)));
    const bf16x4 r4 = __builtin_bit_cast(bf16x4, r);
    va[4 * C + 0] = r4[0];
    va[4 * C + 1] = r4[1];
    va[4 * C + 2] = r4[2];
    va[4 * C + 3] = r4[3];
}
__device__ __forceinline__ bf16x8 load_v_operand(const unsigned char* Vs, int db, int l16, int lg) {
    bf16x8 va;
    load_v_half<0>(va, Vs, db, l16, lg);
    load_v_half<1>(va, Vs, db, l16, lg);
    return va;
}

// The vector ALUs are the scarce resource of the pipeline: next to one MFMA the wavefront
// can issue one exponential, or two plain vector instructions, without delaying the next
// MFMA.  Region 1 therefore exponentiates only the first rows_early<MB>() row blocks; the
// last ("late") row block's probabilities are computed one region earlier, in region 2,
// whose other vector work (the maximum scan) leaves slots free.
template <int MB> constexpr int rows_early() { return MB >= 2 ? MB - 1 : MB; }
// The two pipeline regions share a ring of four MFMA operand buffers.  Operand g of a region
// (eight per region) lives in ring[g & 3] and is read from LDS read_ahead<MB>() groups before
// its MFMAs; the last groups of a region read the first operands of the region that follows
// (K after V after K ...), so the LDS latency never shows at a region's start.  The exception
// is the first region of a stage (FIRST): the stage is only known to have landed after the
// barrier in front of it, so it reads its own first operands and the region before it (LAST)
// reads nothing ahead.
// How many groups (of MB MFMAs, 16.4 cycles each) an operand is read from LDS ahead of its use: three
// is the most the ring allows.  Time of a call with three against two, over shapes of each number of row
// blocks, same box, in turn: one 0.981 to 0.995, two 0.985 to 1.002, three 0.996 to 1.018, four 0.999 to 1.005,
// five 0.996 to 1.000 (and the whole 32K round 64.5 against 64.9 us); four to eight groups with a larger
// ring give no more.
template <int MB> constexpr int read_ahead() { return MB == 3 ? 2 : 3; }

// Pipeline region 1: the matrix cores compute the exponents of the NEXT sub-tile
// (X^T = K Q'^T - m_ref into xn) while the vector ALUs turn the CURRENT sub-tile's exponents
// xc into probabilities (pb, packed bf16) for the early row blocks.  One MFMA and one
// exponential per slot; sched_barrier pins the interleaving because the wavefront issues in
// order.
template <int MB, bool FIRST>
__device__ __forceinline__ void region_qk_exp(const unsigned char* __restrict__ Ks,
                                              const unsigned char* __restrict__ Vnext, const WaveRows<MB>& w,
                                              floatx4 (&xn)[MB][2], const floatx4 (&xc)[MB][2],
                                              uintx4 (&pb)[MB], bf16x8 (&ring)[4], int lane) {
    constexpr int E = rows_early<MB>();
    constexpr int PF = read_ahead<MB>();
    const int l16 = lane & 15, lg = lane >> 4;
    constexpr bool LATE = E < MB;
    constexpr int H = (E + 1) / 2;
    // Exponentials waiting to be packed.  Pair p = groups 2p (-> e0[p & 1]) and 2p + 1 (-> e1).
    // With a late row block its slots do the packing, two per slot so that no slot holds more
    // than 8 cycles of vector work: rows < H of pair p in group 2p + 1, the others in group
    // 2p + 2 (hence two copies of e0).  Without one, a pair is packed next to the exponential
    // one group later.
    float e0[2][E], e1[E];
    if constexpr (FIRST) {
        ring[0] = load_k_operand(Ks, 0, l16, lg);
        ring[1] = load_k_operand(Ks, 1, l16, lg);
        if constexpr (PF > 2) ring[2] = load_k_operand(Ks, 2, l16, lg);
    }
    static_for<0, 8>([&](auto g_) {
        GRAFT_CONST(g, g_);
        constexpr int c = g >> 2, ds = g & 3;
        if constexpr (g + PF < 8) ring[(g + PF) & 3] = load_k_operand(Ks, g + PF, l16, lg);
        else ring[(g + PF) & 3] = load_v_operand(Vnext, g + PF - 8, l16, lg);
        static_for<0, MB>([&](auto rb_) {
            GRAFT_CONST(rb, rb_);
            constexpr bool guard = (g == 0 && rb == 0);
            if constexpr (ds == 0) mfma_x_first<q_reg<MB>(rb, 0), guard>(xn[rb][c], ring[g & 3], w.negm[rb]);
            else mfma_x_next<q_reg<MB>(rb, ds), guard>(xn[rb][c], ring[g & 3]);
            if constexpr (rb < E) {
                if constexpr (!LATE && (g & 1) == 0 && g >= 2)
                    pb[rb][(g - 2) >> 1] = pack_bf16(e0[((g - 2) >> 1) & 1][rb], e1[rb]);
                const float pe = __builtin_amdgcn_exp2f(xc[rb][c][ds]);
                if constexpr (g & 1) e1[rb] = pe;
                else e0[(g >> 1) & 1][rb] = pe;
            } else if constexpr (g & 1) {           // late slot of group 2p + 1: rows < H of pair p
                constexpr int pr = g >> 1;
#pragma unroll
                for (int r = 0; r < H; ++r) pb[r][pr] = pack_bf16(e0[pr & 1][r], e1[r]);
            } else if constexpr (g >= 2) {          // late slot of group 2p + 2: the other rows of pair p
                constexpr int pr = (g - 2) >> 1;
#pragma unroll
                for (int r = H; r < E; ++r) pb[r][pr] = pack_bf16(e0[pr & 1][r], e1[r]);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    });
#pragma unroll
    for (int rb = LATE ? H : 0; rb < E; ++rb) pb[rb][3] = pack_bf16(e0[1][rb], e1[rb]);
    __builtin_amdgcn_sched_barrier(0);
}

// Probabilities of the late row block from its exponents, outside the pipeline: after the
// exponents were changed behind region 2's back (ancestor masking, a new reference).
template <int MB>
__device__ __forceinline__ void late_probabilities(const floatx4 (&x)[MB][2], uintx4& pl) {
    if constexpr (rows_early<MB>() < MB) {
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const float p0 = __builtin_amdgcn_exp2f(x[MB - 1][e >> 2][e & 3]);
            const float p1 = __builtin_amdgcn_exp2f(x[MB - 1][e >> 2][(e & 3) + 1]);
            pl[e >> 1] = pack_bf16(p0, p1);
        }
    }
}

// Pipeline region 2: the matrix cores run O^T += V^T P^T and the row sums of the CURRENT
// sub-tile (probabilities: pb for the early row blocks, pl_cur for the late one) while the
// vector ALUs scan the NEXT sub-tile's exponents xn for their lane-local maxima (first half
// of the region) and turn the late row block's into probabilities pl_next (second half;
// speculative: the caller redoes them when the scan or the masking changes the exponents).
// Returns whether any lane saw an exponent above its row's threshold (wavefront-uniform).
template <int MB, bool LAST>
__device__ __forceinline__ bool region_pv_max(const unsigned char* __restrict__ Vs,
                                              const unsigned char* __restrict__ Knext, WaveRows<MB>& w,
                                              const uintx4 (&pb)[MB], const uintx4& pl_cur, uintx4& pl_next,
                                              const floatx4 (&xn)[MB][2], const bf16x8& ones, float ninf,
                                              float (&lm)[MB], bf16x8 (&ring)[4], int lane) {
    constexpr int E = rows_early<MB>();
    constexpr int PF = read_ahead<MB>();
    constexpr bool LATE = E < MB;
    constexpr bool INLOOP = LATE && MB >= 3;     // three free slots per group are needed
    const int l16 = lane & 15, lg = lane >> 4;
    float le0 = 0.f, le1 = 0.f;
    unsigned long long above = 0;
    static_for<0, 8>([&](auto db_) {
        GRAFT_CONST(db, db_);
        static_for<0, MB>([&](auto rb_) {
            GRAFT_CONST(rb, rb_);
            if constexpr (rb < E) mfma_o<o_reg(rb, db), (db == 0 && rb == 0)>(ring[db & 3], pb[rb]);
            else mfma_o<o_reg(rb, db), (db == 0 && rb == 0)>(ring[db & 3], pl_cur);
            // The slot's vector work, at most 8 cycles of it where the slots suffice.
            // LDS reads of the operand read_ahead<MB>() groups ahead: one half in each of the first two slots.
            if constexpr (rb == 0) {
                if constexpr (db + PF < 8) load_v_half<0>(ring[(db + PF) & 3], Vs, db + PF, l16, lg);
                else if constexpr (!LAST) ring[(db + PF) & 3] = load_k_operand(Knext, db + PF - 8, l16, lg);
            }
            if constexpr (rb == (MB > 1 ? 1 : 0) && db + PF < 8) load_v_half<1>(ring[(db + PF) & 3], Vs, db + PF, l16, lg);
            if constexpr (db < 4) {
                // maximum scan, two exponents of one row block per instruction; slot 0 is left
                // to the LDS read where there are five slots (row blocks 0 and 1 go to slots 1, 2)
                static_for<0, MB>([&](auto r_) {
                    GRAFT_CONST(r, r_);
                    constexpr int slot = MB == 5 ? (r == 0 ? 1 : (r == 1 ? 2 : r)) : r;
                    if constexpr (slot == rb) {
                        const float a = xn[r][db >> 1][2 * (db & 1)], b = xn[r][db >> 1][2 * (db & 1) + 1];
                        // (the three-operand form also for the first pair: a plain two-operand
                        // maximum would first canonicalise both inputs, two more instructions)
                        lm[r] = __builtin_fmaxf(__builtin_fmaxf(db == 0 ? ninf : lm[r], a), b);
                    }
                });
            }
            if constexpr (db == 4 && rb == (MB >= 4 ? 0 : MB - 1)) {
                // the scan is complete: one compare for all row blocks, long before the branch on
                // it at the end of the region (a branch on a fresh vector compare would stall)
                float lmax = lm[0];
#pragma unroll
                for (int r = 1; r < MB; ++r) lmax = __builtin_fmaxf(lmax, lm[r]);
                above = __builtin_amdgcn_ballot_w64(lmax > w.thr_min);
                asm volatile("" : "+s"(above));
            }
            if constexpr (db < 4) {
            } else if constexpr (INLOOP && (rb == MB - 3 || rb == MB - 2)) {
                // late row block: element 2 (db - 4) + {0, 1} of its 8; the pair is packed in
                // the slot after its second exponential
                constexpr int e = 2 * (db - 4) + (rb - (MB - 3));
                const float pe = __builtin_amdgcn_exp2f(xn[MB - 1][e >> 2][e & 3]);
                if constexpr (rb == MB - 3) le0 = pe;
                else le1 = pe;
            } else if constexpr (INLOOP && rb == MB - 1) {
                pl_next[db - 4] = pack_bf16(le0, le1);
                // (pinned here: the caller overwrites pl_next on some paths, and the compiler
                //  would otherwise move these exponentials to the paths that do not)
                asm volatile("" : "+v"(pl_next[db - 4]));
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    });
    if constexpr (LATE && !INLOOP) late_probabilities<MB>(xn, pl_next);
    static_for<0, MB>([&](auto rb_) {
        GRAFT_CONST(rb, rb_);
        if constexpr (rb >= L_IN_ACC) mfma_rowsum(w.lsum_v, ones, rb < E ? pb[rb] : pl_cur);
        else if constexpr (rb < E) mfma_rowsum_acc<l_reg<MB>(rb)>(ones, pb[rb]);
        else mfma_rowsum_acc<l_reg<MB>(rb)>(ones, pl_cur);
    });
    const bool any = above != 0;
#pragma unroll
    for (int rb = 0; rb < E; ++rb) GRAFT_KEEP(pb[rb]);
    GRAFT_KEEP(pl_cur);
    return any;
}

// Ancestor masking of an exponent tile that reaches past the prefix (tree slots and the
// tail): masked entries become -inf; the lane-local maxima are recomputed.
template <int MB>
__device__ __forceinline__ bool apply_tree_mask(floatx4 (&x)[MB][2], const WaveRows<MB>& w, float (&lm)[MB],
                                                int lane, int t_sub0, int P, int n, int slots, int r_base, int R, int g_magic,
                                                const unsigned* __restrict__ Ms) {
    const int l16 = lane & 15, lg = lane >> 4;
    bool grow = false;
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
        const int r = r_base + rb * 16 + l16;
        const int node = (r * g_magic) >> 16;              // r / G
        const unsigned* row = Ms + 4 * (r < R && node < n ? node : 0);     // (rows of absent nodes: any finite mask will do)
        const unsigned win = visible_window(t_sub0 - P, slots, [&](int k) { return row[k]; }) >> (4 * lg);
        reserve_acc_registers<MB>();                          // no temporaries of the compiler's in the accumulators
        float mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[rb][c][i] = keep_visible(x[rb][c][i], win, 16 * c + i);
                mx = fmaxf(mx, x[rb][c][i]);
            }
        lm[rb] = mx;
        grow = grow || (mx > w.thr[rb]);
    }
    return __builtin_amdgcn_ballot_w64(grow) != 0;
}

// Some lane saw an exponent above its row's threshold.  Rows without a reference take the
// tile's row maximum as their reference: nothing has been accumulated for them yet, so only
// the pending exponents are re-based.  Returns true when a row that already has a reference
// exceeded the lazy bound: the caller then leaves the fast loop (that needs a rescale of O).
template <int MB>
__device__ __forceinline__ bool set_references(float (&lm)[MB], WaveRows<MB>& w, floatx4 (&x)[MB][2]) {
    bool raise = false;
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
        float mx = lm[rb];
        mx = rows_max_f32(mx);
        lm[rb] = mx;                                      // now the row maximum, same in the row's 4 lanes
        raise = raise || (!w.unset(rb) && mx > w.thr[rb]);
    }
    if (__builtin_amdgcn_ballot_w64(raise) != 0) return true;
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
        if (w.unset(rb) && lm[rb] > -INFINITY) {
            w.negm[rb] = floatx4{-lm[rb], -lm[rb], -lm[rb], -lm[rb]};
            w.thr[rb] = AT_LAZY_LOG2;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i) x[rb][c][i] -= lm[rb];
        }
    }
    float tm = w.thr[0];
#pragma unroll
    for (int rb = 1; rb < MB; ++rb) tm = fminf(tm, w.thr[rb]);
    w.thr_min = tm;
    return false;
}

// Slow path (exact running max, classic online softmax): raise every row's reference to
// the maximum seen so far, rescaling O and the row sums.  lm holds the row maxima of x.
template <int MB>
__device__ __forceinline__ void raise_references(const float (&lm)[MB], WaveRows<MB>& w, floatx4 (&x)[MB][2]) {
    GRAFT_MFMA_SETTLE();
    static_for<0, MB>([&](auto rb_) {
        GRAFT_CONST(rb, rb_);
        const float mx = lm[rb];
        const bool unset = w.unset(rb);
        const bool move = (!unset && mx > 0.0f) || (unset && mx > -INFINITY);
        if (__builtin_amdgcn_ballot_w64(move) != 0) {
            // rows that do not move get a = 1 and a zero shift
            const float shift = move ? mx : 0.0f;
            const float a = move ? (unset ? 0.0f : __builtin_amdgcn_exp2f(-mx)) : 1.0f;
            if (move) {
                const float nm = (unset ? 0.0f : w.negm[rb][0]) - mx;
                w.negm[rb] = floatx4{nm, nm, nm, nm};
                w.thr[rb] = AT_LAZY_LOG2;
            }
            if constexpr (rb >= L_IN_ACC) w.lsum_v *= a;
            else
                static_for<0, 4>([&](auto k_) {
                    GRAFT_CONST(k, k_);
                    acc_scale<l_reg<MB>(rb) + k>(a);
                });
            static_for<0, 32>([&](auto k_) {
                GRAFT_CONST(k, k_);
                acc_scale<32 * rb + k>(a);
            });
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i) x[rb][c][i] -= shift;
        }
    });
    GRAFT_MFMA_SETTLE();
}

// Slow-path building blocks: the same arithmetic as the pipeline regions, one thing at a time.
template <int MB>
__device__ __forceinline__ void qk_only(const unsigned char* __restrict__ Ks, const WaveRows<MB>& w,
                                        floatx4 (&x)[MB][2], int lane) {
    const int l16 = lane & 15, lg = lane >> 4;
    static_for<0, 8>([&](auto g_) {
        GRAFT_CONST(g, g_);
        const bf16x8 ka = load_k_operand(Ks, g, l16, lg);
        static_for<0, MB>([&](auto rb_) {
            GRAFT_CONST(rb, rb_);
            if constexpr ((g & 3) == 0) mfma_x_first<q_reg<MB>(rb, 0), true>(x[rb][g >> 2], ka, w.negm[rb]);
            else mfma_x_next<q_reg<MB>(rb, (g & 3)), true>(x[rb][g >> 2], ka);
            asm volatile("s_nop 7" ::: "memory");
        });
        asm volatile("s_nop 15" ::: "memory");
        GRAFT_KEEP(ka);
    });
    GRAFT_MFMA_SETTLE();
}
template <int MB>
__device__ __forceinline__ void exp_only(const floatx4 (&x)[MB][2], uintx4 (&pb)[MB]) {
#pragma unroll
    for (int rb = 0; rb < MB; ++rb)
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const float p0 = __builtin_amdgcn_exp2f(x[rb][e >> 2][e & 3]);
            const float p1 = __builtin_amdgcn_exp2f(x[rb][e >> 2][(e & 3) + 1]);
            pb[rb][e >> 1] = pack_bf16(p0, p1);
        }
}
template <int MB>
__device__ __forceinline__ void pv_only(const unsigned char* __restrict__ Vs, WaveRows<MB>& w,
                                        const uintx4 (&pb)[MB], const bf16x8& ones, int lane) {
    const int l16 = lane & 15, lg = lane >> 4;
    static_for<0, 8>([&](auto db_) {
        GRAFT_CONST(db, db_);
        const bf16x8 va = load_v_operand(Vs, db, l16, lg);
        static_for<0, MB>([&](auto rb_) {
            GRAFT_CONST(rb, rb_);
            mfma_o<o_reg(rb, db), true>(va, pb[rb]);
            asm volatile("s_nop 7" ::: "memory");
        });
        asm volatile("s_nop 15" ::: "memory");
        GRAFT_KEEP(va);
    });
    static_for<0, MB>([&](auto rb_) {
        GRAFT_CONST(rb, rb_);
        if constexpr (rb >= L_IN_ACC) mfma_rowsum<true>(w.lsum_v, ones, pb[rb]);
        else mfma_rowsum_acc<l_reg<MB>(rb), true>(ones, pb[rb]);
        asm volatile("s_nop 7" ::: "memory");
    });
    GRAFT_MFMA_SETTLE();
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) GRAFT_KEEP(pb[rb]);
}

// One split only: O / l as bf16, straight from the accumulators.  Lane (l16, lg) holds row l16 of
// each row block, dims 16 db + 4 lg .. +3 of dim block db.  Rows of absent nodes are zeros.
template <int MB>
__device__ __forceinline__ void store_rows(const AttnParams& p, const WaveRows<MB>& w, int b, int g, int r_base,
                                           int n, int lane) {
    const int l16 = lane & 15, lg = lane >> 4;
    static_for<0, MB>([&](auto rb_) {
        GRAFT_CONST(rb, rb_);
        const int r = r_base + rb * 16 + l16;
        float l;
        if constexpr (rb >= L_IN_ACC) l = w.lsum_v[0];
        else l = acc_get<l_reg<MB>(rb)>();
        const int i = (r * p.g_magic) >> 16, hl = r - i * p.G;                  // i = r / G
        const bool keep = i < n && l > 0.f;
        const float inv_l = keep ? 1.0f / l : 0.f;
        unsigned short* outp = static_cast<unsigned short*>(p.out) +
            ((static_cast<int64_t>(b) * p.K_max + i) * p.Hq + g * p.G + hl) * AT_D + 4 * lg;
        static_for<0, 8>([&](auto db_) {
            GRAFT_CONST(db, db_);
            float o[4];
            static_for<0, 4>([&](auto k_) {
                GRAFT_CONST(k, k_);
                const float v = acc_get<o_reg(rb, db) + k>();
                o[k] = keep ? v * inv_l : 0.f;
            });
            if (r < p.R) *reinterpret_cast<uint2*>(outp + 16 * db) = uint2{pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3])};
        });
    });
}

template <int MB>
__global__ __launch_bounds__(AT_THREADS) void tree_attn_mfma_kernel(GRAFT_ATTN_ARGS) {
    __shared__ __attribute__((aligned(1024))) unsigned char kv[AT_NBUF][AT_STAGE_BYTES];
    __shared__ unsigned Ms[GRAFT_MAX_NODES * GRAFT_MASK_WORDS * 2];   // ancestor masks as 32-bit words
    __shared__ int32_t Tb[AT_MAX_SPLIT_PAGES];                         // this split's block-table entries

    reserve_acc_registers<MB>();
    GRAFT_STAMPS_BEGIN();
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_u = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const WorkItem item = xcd_work_item(n_units, n_row_tiles, row_tiles_magic);
    const bool padding = item.unit < 0;          // of the grid (whole workgroup): it leaves behind the first requests, which
                                                 // a branch in front of them would delay
    const int rt = item.row_tile, unit = padding ? 0 : item.unit;             // unit over B * Hkv * n_splits
    const int bg = div31(unit, splits_magic), split = unit - bg * n_splits;
    const int b = div24(bg, n_kv_heads), g = bg - b * n_kv_heads;

    const int n_raw = scalar_load(n_nodes, b), P_raw = scalar_load(prefix_len, b);
    await_setup_args(p);
    if (padding) return;
    const unsigned kv_base = __builtin_amdgcn_readfirstlane(lds_address(&kv[0][0]));
    constexpr int TILE_ROWS = AT_WAVES * 16 * MB;
    const int r_base = rt * TILE_ROWS + wave_u * (16 * MB);
    // The queries lie in the ring until they are read, in front of the values of buffer 3 (which are cleared below); with four and
    // five row blocks they reach into the buffer of stage 1.
    constexpr unsigned Q_END = AT_NBUF * AT_STAGE_BYTES - AT_STAGE * AT_ROW_BYTES;
    constexpr unsigned Q_OFF = MB <= 3 ? 2 * AT_STAGE_BYTES : Q_END - TILE_ROWS * AT_ROW_BYTES;
    constexpr bool Q_OVER_1 = Q_OFF < 2 * AT_STAGE_BYTES;
    static_assert(Q_OFF >= AT_STAGE_BYTES && Q_OFF + TILE_ROWS * AT_ROW_BYTES <= Q_END, "queries of a tile in the ring");
    request_masks(p, b, Ms, tid, wave_u);
    request_queries<TILE_ROWS>(p, b, g, rt * TILE_ROWS, kv_base + Q_OFF, lane, wave_u);
    __builtin_amdgcn_sched_barrier(0);
    const SplitRange sr = split_range(p, n_raw, P_raw, split, n_splits, splits_magic);
    const int n_st = sr.st1 - sr.st0;
#ifdef GRAFT_ATTN_STAMPS
    asm volatile("" : : "s"(n_st));              // (the stamp is taken when the lengths are there)
#endif
    GRAFT_STAMP(AT_TS_LENGTHS);

    // this split's block-table entries to LDS; the pages of this wavefront's first two stages as scalars: with them the first
    // transfers can be issued without a trip through LDS and a barrier
    const int n_pg = n_st * (AT_STAGE / GRAFT_PAGE_SIZE);
    const int32_t* table = p.block_table + static_cast<size_t>(b) * p.max_pages;
    const int first_pg = sr.st0 * (AT_STAGE / GRAFT_PAGE_SIZE);
    const int last_pg = (sr.total - 1) >> 4;
    int32_t first_pages[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int pg = first_pg + 4 * u + wave_u;
        first_pages[u] = scalar_load(table, (4 * u + wave_u) < n_pg ? (pg < last_pg ? pg : last_pg) : 0);
    }
    for (int u = 0; u < n_pg; u += AT_THREADS) {
        const int pg = first_pg + u + tid;
        load_global_to_lds_b32(table + (pg < last_pg ? pg : last_pg), __builtin_amdgcn_readfirstlane(lds_address(Tb)) + 4 * u + 256 * wave_u);
    }
    GRAFT_STAMP(AT_TS_TABLE_REQ);
    // O^T and the row sums to zero
    WaveRows<MB> w;
    static_for<0, MB>([&](auto rb_) {
        GRAFT_CONST(rb, rb_);
        w.thr[rb] = -INFINITY;
        w.thr_min = -INFINITY;
        w.negm[rb] = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (rb >= L_IN_ACC) w.lsum_v = floatx4{0.f, 0.f, 0.f, 0.f};
        else
            static_for<0, 4>([&](auto k_) {
                GRAFT_CONST(k, k_);
                acc_set<l_reg<MB>(rb) + k>(0.0f);
            });
        static_for<0, 32>([&](auto k_) {
            GRAFT_CONST(k, k_);
            acc_set<32 * rb + k>(0.0f);
        });
    });
    // the first pipeline step multiplies zero probabilities with whatever buffer 3 holds: make it zeros
    for (int k = tid; k < AT_STAGE * AT_ROW_BYTES / 16; k += AT_THREADS)
        reinterpret_cast<uint4*>(&kv[AT_NBUF - 1][AT_STAGE * AT_ROW_BYTES])[k] = uint4{0u, 0u, 0u, 0u};
    GRAFT_STAMP(AT_TS_ZEROED);

    // ---- stage pipeline: stage k (split-local) lives in kv[k & 3]; its loads are issued two
    //      stages ahead.  advance(k) = wait for this wavefront's loads of stage k (the next
    //      stage's stay in flight), meet the others, then start stage k + 2.
    const int last_tok = sr.total - 1;
    // A wavefront moves one page per stage: page 4 * stage + wave, 16 token rows of K and of V,
    // four rows (1 KB) per instruction.  Lane (lg, l16) of instruction j fetches 16-byte chunk
    // l16 of row 4 j + lg; which chunk of the row that is (the XOR swizzle) depends on the lane
    // and on j only, so the lane's byte offsets inside a page are loop-invariant.
    unsigned koff[4], voff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = 4 * j + lg;                                  // token row within the page
        const int kchunk = l16 ^ row;
        const int vchunk = (((l16 >> 1) ^ (row & 7)) << 1) | (l16 & 1);
        const unsigned row_off = static_cast<unsigned>(row) * static_cast<unsigned>(p.token_stride) * 2u;
        koff[j] = row_off + kchunk * 16;
        voff[j] = row_off + vchunk * 16;
    }
    auto issue_page = [&](int k, int page) {
        const unsigned buf = kv_base + (k & (AT_NBUF - 1)) * AT_STAGE_BYTES + wave_u * 4096;
        const int t_page = (sr.st0 + k) * AT_STAGE + 16 * wave_u;   // first token of this wavefront's page
        const int64_t page_off = (static_cast<int64_t>(page) * p.page_stride + static_cast<int64_t>(g) * p.head_stride) * 2;
        const unsigned char* kp = static_cast<const unsigned char*>(p.k) + page_off;
        const unsigned char* vp = static_cast<const unsigned char*>(p.v) + page_off;
        if (t_page + 15 <= last_tok) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                load_global_to_lds_b128(kp, koff[j], buf + j * 1024);
                load_global_to_lds_b128(vp, voff[j], buf + AT_STAGE * AT_ROW_BYTES + j * 1024);
            }
        } else {
            // the page holding the last token, or a page past it (its table entry then repeats
            // the last page): rows past the end re-read the last token, whose values are finite
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = 4 * j + lg;
                int t = t_page + row;
                t = t < last_tok ? t : last_tok;
                const int kchunk = l16 ^ row;
                const int vchunk = (((l16 >> 1) ^ (row & 7)) << 1) | (l16 & 1);
                const unsigned row_off = static_cast<unsigned>(t & 15) * static_cast<unsigned>(p.token_stride) * 2u;
                load_global_to_lds_b128(kp, row_off + kchunk * 16, buf + j * 1024);
                load_global_to_lds_b128(vp, row_off + vchunk * 16, buf + AT_STAGE * AT_ROW_BYTES + j * 1024);
            }
        }
    };
    int next_issue = 0;                          // stages are issued in order, each once
    if (n_st > 0) {
        issue_page(0, first_pages[0]);
        next_issue = 1;
    }
    GRAFT_STAMP(AT_TS_STAGE0_REQ);
    if (!Q_OVER_1 && n_st > 1) {
        issue_page(1, first_pages[1]);
        next_issue = 2;
    }
    // Queries, masks and table are there when only the stages are in flight.  Q' = bf16(Q * scale * log2 e) into AccVGPRs, while the
    // first keys are on their way.
    if (next_issue == 2) GRAFT_WAIT_VMCNT(2 * AT_LOADS_PER_STAGE);
    else if (next_issue == 1) GRAFT_WAIT_VMCNT(AT_LOADS_PER_STAGE);
    else GRAFT_WAIT_VMCNT(0);
    lds_barrier();                               // (LDS only: the transfers stay in flight)
    GRAFT_STAMP(AT_TS_TABLE_LDS);
    const float c_log2 = p.scale_log2e;
    uintx4 qd[MB][4];                            // (all reads in flight)
#pragma unroll
    for (int rb = 0; rb < MB; ++rb)
#pragma unroll
        for (int ds = 0; ds < 4; ++ds)
            qd[rb][ds] = __builtin_bit_cast(uintx4, load_k_operand(&kv[0][0] + Q_OFF + (wave_u * (16 * MB) + rb * 16) * AT_ROW_BYTES, ds, l16, lg));
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, MB>([&](auto rb_) {
        GRAFT_CONST(rb, rb_);
        static_for<0, 16>([&](auto k_) {
            GRAFT_CONST(k, k_);
            acc_set_bits<q_reg<MB>(rb, 0) + k>(scale_bf16_pair(qd[rb][k >> 2][k & 3], c_log2));
        });
    });
    GRAFT_STAMP(AT_TS_Q_DONE);
    if constexpr (Q_OVER_1) {
        lds_barrier();                           // everybody has read
        if (n_st > 1) {
            issue_page(1, first_pages[1]);
            next_issue = 2;
        }
    }

    int tb_next = Tb[2 * 4 + wave_u];            // the next stage's table entry is read one stage early
    auto issue_stage = [&](int k) {
        const int page = __builtin_amdgcn_readfirstlane(tb_next);
        const int nxt = (k + 1) * 4 + wave_u;
        tb_next = Tb[nxt < AT_MAX_SPLIT_PAGES ? nxt : AT_MAX_SPLIT_PAGES - 1];
        issue_page(k, page);
    };
    // arrive(k): wait for this wavefront's transfers of stage k (those of stage k + 1 stay in
    // flight) and meet the other wavefronts.  After it stage k can be read and the buffer of
    // stage k + 2 (last read in step k - 1) can be refilled.  advance(k) also starts stage k + 2.
    auto arrive = [&](int k) {
        GRAFT_SPAN_BEGIN();
        if (k + 1 < n_st) GRAFT_WAIT_VMCNT(AT_LOADS_PER_STAGE);
        else GRAFT_WAIT_VMCNT(0);
        GRAFT_SPAN_SPLIT(AT_TS_WAIT_CYCLES);
        lds_barrier();
        GRAFT_SPAN_END(AT_TS_BARRIER_CYCLES);
    };
    // The compute unit's address path takes about 16 cycles per 1 KB transfer, and a wavefront
    // that issues waits for its turn: four wavefronts issuing their 8 transfers at the same
    // time hold each other up for about 500 cycles.  So only the first two issue right after
    // the barrier; the other two issue in the middle of the stage (the target buffer is free
    // during the whole stage), when the first two are computing.
    const bool early_wave = wave_u < 2;
    auto issue_upto = [&](int s) {
        while (next_issue <= s && next_issue < n_st) issue_stage(next_issue++);
    };
    auto advance = [&](int k) {
        arrive(k);
        if (early_wave) issue_upto(k + 2);
    };

    // Only the transfers of stages 0 and 1 are in flight here, and the first advance() waits
    // for stage 0 alone.
    GRAFT_MFMA_SETTLE();

    uintx4 ones_bits;
#pragma unroll
    for (int t = 0; t < 4; ++t) ones_bits[t] = opaque_bits(0x3f803f80u);    // 1.0 in both bf16 halves
    const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_bits);
    constexpr int K_OFF = 0, V_OFF = AT_STAGE * AT_ROW_BYTES, SUB = AT_SUB * AT_ROW_BYTES;

    // ---- fast loop, software pipelined over 32-token sub-tiles.  Step j: region 1 computes
    //      the exponents of sub-tile j while exponentiating sub-tile j-1 (-> pb); region 2
    //      accumulates P.V and the row sums of sub-tile j-1 while scanning the maxima of
    //      sub-tile j.  Exponents ping-pong between xa (even j) and xb (odd j).  The first
    //      step exponentiates -inf (zero probabilities against the zero-filled buffer 3), the
    //      last (drain) step computes exponents nobody uses.  A row's reference is the row
    //      maximum of the first tile that gives it a finite score and is kept while later
    //      exponents stay below AT_LAZY_LOG2; otherwise the wavefront leaves for the slow loop
    //      below (exact running max, rescaling O with the vector ALUs).
    floatx4 xa[MB][2], xb[MB][2];
    uintx4 pb[MB];
    uintx4 pla = uintx4{0u, 0u, 0u, 0u}, plb = pla;   // late row block's probabilities: even / odd sub-tiles
    float lm[MB];
    const float ninf = __uint_as_float(opaque_bits(0xff800000u));
    bf16x8 ring[4];            // MFMA operands read ahead from LDS (see the regions)
#pragma unroll
    for (int rb = 0; rb < MB; ++rb)
#pragma unroll
        for (int c = 0; c < 2; ++c) xb[rb][c] = floatx4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};

    GRAFT_STAMP(AT_TS_LOOP);
    GRAFT_STAMP_CYCLES(AT_TS_CYCLES_LOOP);
    const int n_sub = 2 * n_st;
    int j = 0;                 // sub-tile whose exponents are pending when the fast loop is left
    bool slow = false;
    for (int k = 0; k <= n_st; ++k) {
        reserve_acc_registers<MB>();    // nothing of the compiler's may live in the hand-managed AccVGPRs here
        const bool live = k < n_st;
        // (transfers of stage k + 2: see advance(); issuing them inside the MFMA regions was
        //  measured slower, a transfer issued while MFMAs are in flight stalls the wavefront)
        if (live) advance(k);
#ifdef GRAFT_ATTN_STAMPS
        if (k == 0) GRAFT_STAMP(AT_TS_STAGE0);
#endif
        const unsigned char* cur = kv[k & (AT_NBUF - 1)];
        const unsigned char* prev = kv[(k - 1) & (AT_NBUF - 1)];
        const int t0 = (sr.st0 + k) * AT_STAGE;
        // even sub-tile of stage k
        // (the late row block's probabilities of the odd sub-tile before, plb, are consumed
        //  while those of this even sub-tile, pla, are produced; and the other way round below)
        region_qk_exp<MB, true>(cur + K_OFF, prev + V_OFF + SUB, w, xa, xb, pb, ring, lane);
        bool grow = region_pv_max<MB, false>(prev + V_OFF + SUB, cur + K_OFF + SUB, w, pb, plb, pla, xa, ones, ninf, lm, ring, lane);
        if (!live) break;
        // (where the exponents change after region 2 has turned the late row block's into
        //  probabilities, those are redone)
        if (__builtin_expect(t0 + AT_SUB > sr.P, 0)) {
            grow = apply_tree_mask<MB>(xa, w, lm, lane, t0, sr.P, sr.n, sr.total - sr.P, r_base, p.R, p.g_magic, Ms);
            late_probabilities<MB>(xa, pla);
        }
        if (__builtin_expect(grow, 0)) {
            if (set_references<MB>(lm, w, xa)) { slow = true; j = 2 * k; break; }
            late_probabilities<MB>(xa, pla);
        }
        if (!early_wave) issue_upto(k + 2);
        // odd sub-tile of stage k
        region_qk_exp<MB, false>(cur + K_OFF + SUB, cur + V_OFF, w, xb, xa, pb, ring, lane);
        grow = region_pv_max<MB, true>(cur + V_OFF, nullptr, w, pb, pla, plb, xb, ones, ninf, lm, ring, lane);
        if (__builtin_expect(t0 + 2 * AT_SUB > sr.P, 0)) {
            grow = apply_tree_mask<MB>(xb, w, lm, lane, t0 + AT_SUB, sr.P, sr.n, sr.total - sr.P, r_base, p.R, p.g_magic, Ms);
            late_probabilities<MB>(xb, plb);
        }
        if (__builtin_expect(grow, 0)) {
            if (set_references<MB>(lm, w, xb)) {
                slow = true;
                j = 2 * k + 1;
#pragma unroll
                for (int rb = 0; rb < MB; ++rb)
#pragma unroll
                    for (int c = 0; c < 2; ++c) xa[rb][c] = xb[rb][c];
                break;
            }
            late_probabilities<MB>(xb, plb);
        }
    }

    // ---- slow loop (rare): xa holds the exponents of sub-tile j against the old references and
    //      lm their row maxima.  One sub-tile at a time, exact running max.
    if (slow) {
        issue_upto((j >> 1) + 2);       // a late-issuing wavefront may have left before its turn
        while (true) {
            reserve_acc_registers<MB>();
            const unsigned char* cur = kv[(j >> 1) & (AT_NBUF - 1)] + (j & 1) * SUB;
            raise_references<MB>(lm, w, xa);
            exp_only<MB>(xa, pb);
            pv_only<MB>(cur + V_OFF, w, pb, ones, lane);
            ++j;
            if (j >= n_sub) break;
            if ((j & 1) == 0) {
                advance(j >> 1);
                issue_upto((j >> 1) + 2);
            }
            qk_only<MB>(kv[(j >> 1) & (AT_NBUF - 1)] + (j & 1) * SUB + K_OFF, w, xa, lane);
#pragma unroll
            for (int rb = 0; rb < MB; ++rb) {
                float mx = -INFINITY;
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) mx = fmaxf(mx, xa[rb][c][i]);
                lm[rb] = mx;
            }
            const int t_sub0 = sr.st0 * AT_STAGE + j * AT_SUB;
            if (t_sub0 + AT_SUB > sr.P)
                apply_tree_mask<MB>(xa, w, lm, lane, t_sub0, sr.P, sr.n, sr.total - sr.P, r_base, p.R, p.g_magic, Ms);
#pragma unroll
            for (int rb = 0; rb < MB; ++rb) {
                float mx = lm[rb];
                mx = fmaxf(mx, __shfl_xor(mx, 16));
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                lm[rb] = mx;
            }
        }
    }
    GRAFT_MFMA_SETTLE();
    GRAFT_STAMP(AT_TS_LOOP_END);
    GRAFT_STAMP_CYCLES(AT_TS_CYCLES_END);

    if (n_splits == 1) {
        // ---- one split: this workgroup holds the whole result of its rows
        // (the lane index goes through an empty asm: otherwise the compiler keeps the row
        //  addressing it computed for the Q loads in registers across the whole loop, registers
        //  that the loop does not have)
        int lane_out = lane;
        asm volatile("" : "+v"(lane_out));
        store_rows<MB>(p, w, b, g, r_base, sr.n, lane_out);
        GRAFT_STAMPS_WRITE(p, n_st);
        return;
    }
    // ---- partial results.  Per row and split: the reference max m (log2 units), the row sum l
    //      and O / l, which is a convex combination of V rows, stored as fp16 after an exact
    //      scaling by a power of two 2^-e that brings the row's largest magnitude into
    //      [0.5, 1): eleven significant bits relative to the row's largest entry, eight times
    //      finer than the bf16 rounding of the final output, at half the bytes of fp32 for the
    //      round trip through memory that the splits cost.  The rows are written as the
    //      accumulator tiles lie in the registers (two 16 x 16 tiles side by side, 16 bytes per
    //      lane), so that every store instruction fills 1 KB of consecutive addresses.
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
    const size_t part = ((static_cast<size_t>(b) * n_kv_heads + g) * n_splits + split) * p.R_pad;
    static_for<0, MB>([&](auto rb_) {
        GRAFT_CONST(rb, rb_);
        const int r0 = r_base + rb * 16;                          // first row of this 16-row block
        float l;
        if constexpr (rb >= L_IN_ACC) l = w.lsum_v[0];
        else l = acc_get<l_reg<MB>(rb)>();
        const float inv_l = l > 0.f ? 1.0f / l : 0.f;
        float ov[32];
        static_for<0, 32>([&](auto k_) {
            GRAFT_CONST(k, k_);
            ov[k] = acc_get<o_reg(rb, 0) + k>();
        });
        float amax = 0.f;
#pragma unroll
        for (int k = 0; k < 32; ++k) amax = fmaxf(amax, fabsf(ov[k]));
        amax = rows_max_f32(amax);                                // the row's, same in its four lanes
        // biased exponent of the normalised row maximum, kept where 2^e and 2^-e are normal numbers
        // (a zero row, or values at the ends of the fp32 range, keep a scale they can live with)
        int ex = static_cast<int>((__float_as_uint(amax * inv_l) >> 23) & 0xffu);
        ex = ex < 2 ? 126 : (ex > 252 ? 252 : ex);
        const float pow2e = __uint_as_float(static_cast<unsigned>(ex + 1) << 23);      // 2^(ex - 126)
        const float f = inv_l * __uint_as_float(static_cast<unsigned>(253 - ex) << 23);  // 2^-(ex - 126) / l
        unsigned short* op = p.ws_o + (part + r0) * AT_D + 8 * lane;
        static_for<0, 4>([&](auto dp_) {
            GRAFT_CONST(dp, dp_);
            uintx4 t;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                t[k] = __builtin_bit_cast(unsigned, __builtin_convertvector(
                           floatx2{ov[8 * dp + 2 * k] * f, ov[8 * dp + 2 * k + 1] * f}, halfx2));
            *reinterpret_cast<uintx4*>(op + 512 * dp) = t;
        });
        if (lg == 0)
            *reinterpret_cast<floatx4*>(p.ws_ml + (part + r0 + l16) * 4) = floatx4{w.m_ref(rb), l, pow2e, 0.f};
    });
    GRAFT_STAMPS_WRITE(p, n_st);
}

// Merge the splits of two adjacent 16-row x 16-dim output tiles:
// out = sum_s w_s l_s 2^e_s o_s / sum_s w_s l_s with w_s = 2^(m_s - max m), o_s the stored
// fp16 rows.  Lane (l16, lg) owns row l16, dims 4 lg .. +3 of both tiles, exactly the 16 bytes
// it wrote of every split's block, so a split is one 1 KB read per wavefront.  The kernel is
// a chain of memory round trips, not a stream, so a wavefront takes at most U splits (U = 2,
// 4, 8, 12 or 16, the smallest that covers them: registers, and the instructions, which are cold
// here, go with U) and has all their loads in flight at once (a split without keys has
// weight 0 and a zero block); with more than 16 splits, up to four wavefronts share a tile
// pair and the first of them merges their sums through LDS.
// All loads at once needs buffer loads, which return zeros behind the last split: with a condition
// around every pair the first one was waited for in front of the second.  Requested with the
// arguments that only the end needs, and without the divisions in front: 32 layers of 2K keys
// (9 splits) 430 -> 408 us a round (404 -> 395 of it from 12 splits' loads instead of 16), one of
// 32K keys (31 splits) 65.6 -> 63.9.  Two splits of 8 sequences of 4K keys take 5.8 us either way, and
// with four tile pairs a wavefront: there it is 19 MB through the Infinity Cache.
// WIDE: the partial rows of tree_attn_wide_kernel, in blocks of 32 rows x 16 dims.
constexpr int CB_MAX_SPLITS = 16;
constexpr int CB_MAX_WAVES = 8;          // per workgroup; the host picks a multiple of the wavefronts per tile pair

// shape: wavefronts per tile pair, tile pairs per workgroup (8 bits each), ceil(256 / the former) (9 bits), and the shift of the magic_any of
// the row blocks of a (b, g), at most 140 of them; n_blk_magic: its multiplier.
template <int U, bool WIDE>
__global__ __launch_bounds__(64 * CB_MAX_WAVES) void tree_attn_combine_kernel(
    const unsigned short* ws_o, const float* ws_ml, const int32_t* n_nodes, int32_t n_tiles, int32_t shape, int32_t R, int32_t R_pad,
    int32_t n_splits, uint32_t n_blk_magic, int32_t n_kv_heads, AttnParams p) {
    typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
    // (m, den, acc[8]) per lane of the helper wavefronts (only U = 16 has helpers)
    __shared__ float xch[U == CB_MAX_SPLITS ? CB_MAX_WAVES : 1][10][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wpt = shape & 255, tiles_per_wg = shape >> 8 & 255, pair = wave * (shape >> 16 & 511) >> 8;      // wave / wpt
    constexpr int BLK = WIDE ? 32 : 16, PIECES = AT_D * BLK / 512;          // rows of a block, tile pairs in it
    const int lr = lane % BLK, lg = lane / BLK;
    const int n_blk = R_pad / BLK;                                          // row blocks per (b, g)
    const int tile = static_cast<int>(blockIdx.x) * tiles_per_wg + pair;         // over B*Hkv*n_blk*PIECES
    const int tile_c = tile < n_tiles ? tile : 0;
    const int part_i = wave - pair * wpt;                                        // which U splits
    const int dp = static_cast<unsigned>(tile_c) % PIECES;                                              // dims 32 dp .. 32 dp + 31 (WIDE: 16 dp ..)
    const int bg = div_any(tile_c / PIECES, n_blk_magic, shape >> 25), blk = tile_c / PIECES - bg * n_blk;   // b * Hkv + g, row block
    const int r = blk * BLK + lr;
    const bool live = tile < n_tiles && r < R;                              // not a padding row or tile
    const int s0 = part_i * U;

    // the rows of a (b, g), all splits: what lies behind the last one is read as zeros
    const unsigned rows = tile < n_tiles ? static_cast<unsigned>(n_splits) * R_pad : 0u;
    const size_t row0 = static_cast<size_t>(bg) * n_splits * R_pad;
    const auto o_rows = merge_buffer(ws_o + row0 * AT_D, rows * (AT_D * 2)), ml_rows = merge_buffer(ws_ml + row0 * 4, rows * 16);
    const unsigned ml_at = (s0 * R_pad + r) * 16, o_at = (s0 * R_pad + blk * BLK) * (AT_D * 2) + 1024 * dp + 16 * lane;
    floatx4 ml[U];
    uintx4 ov[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if constexpr (WIDE) {
            ml[u] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(ml_rows, ml_at + u * (R_pad * 16), 0, 0));
        } else {                                // (the fourth number is not used: a register that is free in front of its load is waited for)
            const auto x = __builtin_amdgcn_raw_buffer_load_b96(ml_rows, ml_at + u * (R_pad * 16), 0, 0);
            ml[u] = floatx4{__uint_as_float(x[0]), __uint_as_float(x[1]), __uint_as_float(x[2]), 0.f};
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) ov[u] = __builtin_amdgcn_raw_buffer_load_b128(o_rows, o_at + u * (R_pad * (AT_D * 2)), 0, 0);
    __builtin_amdgcn_sched_barrier(0);                                      // (all of them in flight: the compiler would save registers)
    const int b = div24(bg, n_kv_heads), g = bg - b * n_kv_heads;
    int n = scalar_load(n_nodes, b);                                        // (needed only at the end, like the arguments)
    asm volatile("" : "+s"(n) : "s"(p.out), "s"(p.K_max), "s"(p.Hq), "s"(p.G), "s"(p.g_magic));
    float m_run = -INFINITY, den = 0.f;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (s0 + u >= n_splits) ml[u][0] = -INFINITY;
        m_run = fmaxf(m_run, ml[u][0]);
    }
    float wu[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float wl = ml[u][0] > -INFINITY ? __builtin_amdgcn_exp2f(ml[u][0] - m_run) * ml[u][1] : 0.f;
        den += wl;
        const float low = ml[u][2], high = ml[u][3];                        // (picked by value, not by index)
        wu[u] = wl * (WIDE && dp >= PIECES / 2 ? high : low);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const halfx8 h = __builtin_bit_cast(halfx8, ov[u]);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += wu[u] * static_cast<float>(h[e]);
    }
    if (U == CB_MAX_SPLITS && wpt > 1) {                                      // uniform over the workgroup
        if (part_i > 0) {
            xch[wave][0][lane] = m_run;
            xch[wave][1][lane] = den;
#pragma unroll
            for (int e = 0; e < 8; ++e) xch[wave][2 + e][lane] = acc[e];
        }
        __syncthreads();
        if (part_i > 0) return;
        float m_all = m_run;
        for (int k = 1; k < wpt; ++k) m_all = fmaxf(m_all, xch[wave + k][0][lane]);
        const float keep = m_run > -INFINITY ? __builtin_amdgcn_exp2f(m_run - m_all) : 0.f;
        den *= keep;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= keep;
        for (int k = 1; k < wpt; ++k) {
            const float mk = xch[wave + k][0][lane];
            const float wk = mk > -INFINITY ? __builtin_amdgcn_exp2f(mk - m_all) : 0.f;
            den += wk * xch[wave + k][1][lane];
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += wk * xch[wave + k][2 + e][lane];
        }
    }
    if (!live) return;
    const int i = (r * p.g_magic) >> 16, hl = r - i * p.G;                     // i = r / G
    unsigned short* outp = static_cast<unsigned short*>(p.out) +
        ((static_cast<int64_t>(b) * p.K_max + i) * p.Hq + g * p.G + hl) * AT_D + (WIDE ? 16 * dp + 8 * lg : 32 * dp + 4 * lg);
    if (n < 1 || n > p.K_max) n = 0;
    const float inv = den > 0.f ? 1.0f / den : 0.f;
    unsigned o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        o[k] = pack_bf16(acc[2 * k] * inv, acc[2 * k + 1] * inv);
    if (i >= n) o[0] = o[1] = o[2] = o[3] = 0u;   // rows of absent nodes are zeros whatever their Q rows held
    if constexpr (WIDE) {                         // lanes r and r + 32 have dims 4 lg .. +3 and 8 + 4 lg .. +3: eight in a row for either
        const auto x = __builtin_amdgcn_permlane32_swap(o[0], o[2], false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(o[1], o[3], false, false);
        *reinterpret_cast<uintx4*>(outp) = uintx4{x[0], y[0], x[1], y[1]};
        return;
    }
    *reinterpret_cast<uint2*>(outp) = uint2{o[0], o[1]};          // dims 32 dp + 4 lg .. +3
    *reinterpret_cast<uint2*>(outp + 16) = uint2{o[2], o[3]};     // dims 32 dp + 16 + 4 lg .. +3
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct AttnPlan {
    int mb, n_row_tiles, n_splits, r_pad;       // mb: 64 rows of a tile each
    bool wide;                                  // tree_attn_wide_kernel
    size_t ws_o_bytes, ws_bytes;
    double cost, line;              // estimated cycles; those the direct path is compared with
};

int device_compute_units() {
    static int cached = 0;
    if (cached == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            cached = n;
        else
            cached = 256;
        (void)hipGetLastError();
    }
    return cached;
}

#ifdef GRAFT_ATTN_STAMPS
static thread_local int g_force_splits = 0, g_force_row_tiles = 0;
#endif

// Launch shape of the MFMA path.  One workgroup per compute unit is resident at a time, so
// the job runs in ceil(workgroups / CUs) rounds, each as long as one workgroup's pass: a
// fixed part (set-up, Q conversion, writing the partial results) plus its stages.  The
// numbers are cycles measured on MI355X; the plan takes the row tiling (tiles of 64 mb rows) and the
// number of splits (<= 64, each with at most AT_MAX_SPLIT_PAGES pages) that make the
// estimate smallest.  It depends on the capacity max_pages, not on the actual lengths.
//
// Which kernel: tiles of 64 and 320 rows have the one with 16-row blocks (per stage about 680 mb + 1100, fixed about 3300 mb + 8000), of
// 256 and 384 the one with 32-row blocks, of 128 and 192 either: its loop is faster, its fixed part (twice the rows a wavefront, a merge
// through LDS) longer.  Tiles of 192 rows, time with 32-row blocks over time with 16-row blocks at the same plan, by stages of a split
// (of the geometric mean, over 540 plans of 230 drawn shapes): several splits, under 8 stages 1.03, 8 to 10 1.01, 11 to 13 0.98, 14 to 18
// 0.96, 26 to 40 0.94, above 0.93; one split 1.01, 0.94, 0.95, 0.90, 0.89, 0.86.  Hence the 11 stages.  A sequence with an eighth of the keys its
// table has room for takes 1.0 to 1.1 times as long with 32-row blocks there.
// 256 rows: 5 stages 22.8 / 21.7, 17 43.8 / 43.7, 24 60.6 / 60.5, 63 137.1 / 133.2.  384 rows against two tiles of 192, 16-row
// blocks not offered: 16 for 32 stages 58.8 / 54.6, 128 for 257 365 / 367 (a round 380 / 399 us).  In splits of few stages their partial rows,
// up to two and a half times as many, cost more than the model has: 14 drawn shapes with splits of 5 to 8 stages took 0.97 to 1.18 times
// (geometric mean 1.07) what they took with the 16-row kernel, and take 0.85 to 0.98 times as long in what they get with the 11 stages asked here too.
// 128 rows, two to five row tiles, same plan, by stages of a split: 3 stages 1.08, 5 0.99 to 1.01, 8 0.95, 11 0.92 to 0.94, 14 0.89 to 0.92, 20
// 0.86 to 0.89, 33 0.87, 64 0.81 to 0.93.  One row tile has a stage's keys to itself and is bound by their arrival: 3 to 14 stages 1.00 to
// 1.08, 20 to 64 0.93 to 1.04, so it keeps the 16-row kernel.  So do plans of 64-row tiles, which the larger tile cuts into half as many splits more or twice as many: six shapes take 0.85 to
// 0.90 times as long with it where the table is full, but 0.95 to 1.08 with half the keys and 1.15 to 1.35 with an eighth.  The other 114 of 120
// drawn shapes that get this tile, a third of them in place of one of 256 rows and twice the splits: 0.92 times the time with a full table
// (0.73 .. 1.01), 0.90 with half the keys (0.66 .. 1.01), 0.89 with an eighth (0.53 .. 1.15: dearest where the plan is the same and a
// split of 11 to 17 stages has one or two, 1.06 in 43 shapes: the set-up and exchange of 32-row blocks).
// The best shape of either kernel is found first; between them the launch that merges splits counts, and the 32-row kernel has to
// be ahead by the 3 per cent to which the costs are calibrated.  Tiles of 192 rows that need no split against 320 rows in two:
// 12 stages 24.5 / 31.9 us, 16 29.2 / 35.5 (8 sequences, 80 x 64 heads on 8).
constexpr int WIDE_MIN_STAGES = 11;
struct TileCost { double stage, fixed; };
static TileCost tile_cost(int mb, bool wide) {
    if (!wide) return {680.0 * mb + 1100.0, 3300.0 * mb + 8000.0};
    if (mb == 2) return {2150.0, 14500.0};
    return mb == 3 ? TileCost{2750.0, 19500.0} : (mb == 4 ? TileCost{3650.0, 21000.0} : TileCost{5300.0, 27000.0});
}
static bool has_kernel(int mb, bool wide, int row_tiles, int splits, int64_t stages_per_split) {
    if (!wide) return mb <= 3 || mb == 5;
    const bool enough = stages_per_split >= WIDE_MIN_STAGES;
    return mb == 4 || (mb == 2 && row_tiles > 1 && enough) || (mb == 3 && enough) || (mb == 6 && (splits == 1 || enough));
}
static AttnPlan make_plan(int32_t B, int32_t K_max, int32_t Hq, int32_t Hkv, int32_t max_pages) {
    const int R = K_max * (Hq / Hkv);
    const int rows_per_mb = AT_WAVES * 16;                       // rows a workgroup covers per MB
    const int64_t stages = (static_cast<int64_t>(max_pages) * GRAFT_PAGE_SIZE + AT_STAGE - 1) / AT_STAGE;
    const int64_t min_splits = (stages * (AT_STAGE / GRAFT_PAGE_SIZE) + AT_MAX_SPLIT_PAGES - 1) / AT_MAX_SPLIT_PAGES;
    const int64_t cus = device_compute_units();
    const int s_lo = static_cast<int>(min_splits < 1 ? 1 : min_splits), s_hi = static_cast<int>(stages < 1 ? 1 : (stages < AT_MAX_SPLITS ? stages : AT_MAX_SPLITS));
    int64_t per[AT_MAX_SPLITS + 1];                              // stages of a split
    for (int sp = s_lo; sp <= s_hi; ++sp) per[sp] = (stages + sp - 1) / sp;
    // line: what the direct path is compared with, 16-row blocks only, in tiles of 256 rows too, as when it was measured.  With the costs of
    // what runs now 7 of 4000 shapes (drawn from 1 to 16 sequences of 32 to 64K keys) would change to 32-row blocks without a
    // split: 17.6 .. 24.2 -> 16.1 .. 20.4 us, and an error against 64 bits of 2.35e-3 instead of 2.33e-3.
    struct Best {
        double key = -1.0, cost = 0.0;
        int mb = 0, row_tiles = 0, splits = 0;
    };
    Best narrow, wide, line;
    const auto search = [&](bool w) {
        const int mb_max = w ? 6 : 5;
        const int rt_min = (R + rows_per_mb * mb_max - 1) / (rows_per_mb * mb_max);
        const int rt_max = (R + rows_per_mb - 1) / rows_per_mb;
        for (int rt = rt_min; rt <= rt_max && rt <= rt_min + 3; ++rt) {
            const int mb = (R + rt * rows_per_mb - 1) / (rt * rows_per_mb);
            const TileCost c = tile_cost(mb, w);
            const int64_t units = static_cast<int64_t>(B) * Hkv * rt;
            const double least = c.fixed + c.stage * static_cast<double>(units * stages) / static_cast<double>(cus);    // (all units busy all the time)
            if (narrow.mb > 0 && (w ? least >= 0.97 * narrow.cost : least >= narrow.key && least >= line.key)) continue;
            for (int sp = s_lo; sp <= s_hi; ++sp) {
                const int64_t rounds = (units * sp + cus - 1) / cus;
                const double cost = rounds * (c.fixed + per[sp] * c.stage) + 300.0 * sp;
                const double total = cost + (sp > 1 ? 11500.0 - 200.0 * sp : 0.0);    // with the merge launch, as measured
                const double key = w ? total : cost;
                const auto take = [&](Best& best) {
                    if (best.key < 0.0 || key < best.key) best = {key, total, mb, rt, sp};
                };
                if (has_kernel(mb, w, rt, sp, per[sp]) && !(w && mb == 2 && narrow.mb == 1)) take(w ? wide : narrow);
                if (!w) take(line);
            }
        }
    };
    search(false);
    search(true);
    const bool use_wide = wide.mb > 0 && (narrow.mb == 0 || wide.cost < 0.97 * narrow.cost);
    const Best& best = use_wide ? wide : narrow;
    AttnPlan pl{best.mb, best.row_tiles, best.splits, 0, use_wide, 0, 0, best.cost, line.cost};
#ifdef GRAFT_ATTN_STAMPS
    // timing build: a plan held fixed by the caller (to compare runs that differ in nothing else)
    if (g_force_splits >= (min_splits < 1 ? 1 : min_splits) && g_force_splits <= (stages < AT_MAX_SPLITS ? stages : AT_MAX_SPLITS) && g_force_row_tiles >= 1) {
        const int mb = (R + g_force_row_tiles * rows_per_mb - 1) / (g_force_row_tiles * rows_per_mb);
        const int64_t stages_of_split = (stages + g_force_splits - 1) / g_force_splits;
        if (has_kernel(mb, true, g_force_row_tiles, g_force_splits, stages_of_split) || has_kernel(mb, false, g_force_row_tiles, g_force_splits, stages_of_split)) {
            pl.n_splits = g_force_splits;
            pl.n_row_tiles = g_force_row_tiles;
            pl.mb = mb;
            pl.wide = has_kernel(mb, true, g_force_row_tiles, g_force_splits, stages_of_split);
        }
    }
#endif
    pl.r_pad = pl.n_row_tiles * pl.mb * rows_per_mb;
    if (pl.n_splits > 1) {                                       // one split needs no workspace and no merge
        const size_t rows = static_cast<size_t>(B) * Hkv * pl.n_splits * pl.r_pad;
        pl.ws_o_bytes = rows * AT_D * sizeof(unsigned short);   // fp16 rows
        pl.ws_bytes = pl.ws_o_bytes + rows * 4 * sizeof(float);
    }
    return pl;
}

// Which path, and its plan.  bf16 with D = 128 has two.  Measured, the direct one is faster where one
// launch of it covers the keys (few of them, or many sequences and heads: 6.3 us against 10 to 12 us for
// the MFMA path's two launches) and even with it, within a few per cent, around 2K keys for 8 heads; the
// MFMA path wins from there on, up to 1.5 times on large problems.  Both costs are calibrated to about
// 5 per cent, so the direct path has to be ahead by that much.
struct PathChoice {
    bool direct, only_direct;
    AttnPlan mfma;
    DirectPlan dir;
    DirectPlan unsplit;             // fp32 and D = 64: for callers without a workspace
};
static PathChoice make_choice(int32_t B, int32_t K_max, int32_t Hq, int32_t Hkv, int32_t D, int32_t max_pages, int32_t dtype) {
    PathChoice c{};
    c.dir = plan_direct(B, K_max, Hq, Hkv, D, max_pages, dtype, true);
    if (dtype != GRAFT_BF16 || D != AT_D) {
        c.direct = true;
        c.unsplit = c.dir.n_splits > 1 ? plan_direct(B, K_max, Hq, Hkv, D, max_pages, dtype, false) : c.dir;
        return c;
    }
    c.mfma = make_plan(B, K_max, Hq, Hkv, max_pages);
    // (the MFMA path reads a sequence's queries through a buffer descriptor: less than 4 GB of them)
    c.only_direct = static_cast<int64_t>(K_max) * Hq * AT_ROW_BYTES >= (int64_t{1} << 32);
    c.direct = c.only_direct || c.dir.cost < 0.95 * c.mfma.line;
    return c;
}

// The choices of the last eight shapes are kept per host thread: all layers of a model ask for the same one, a
// draft and a target model or two batch sizes take turns, and working the cost models out takes one to two
// microseconds, a sixth of a small launch (workspace query through ctypes, three shapes with a new table size each time: 2.0
// to 2.5 us; of a kept choice 0.9).  The reference returned is good until the thread's next call.
static const PathChoice& choose_path(int32_t B, int32_t K_max, int32_t Hq, int32_t Hkv, int32_t D, int32_t max_pages, int32_t dtype) {
    struct Kept {
        int32_t key[8];
        PathChoice choice;
    };
    constexpr int KEPT = 8;
    static thread_local Kept kept[KEPT]{};
    static thread_local int last = 0, oldest = 0;
    int32_t key[8] = {B, K_max, Hq, Hkv, D, max_pages, dtype, 1};
#ifdef GRAFT_ATTN_STAMPS
    key[7] += g_force_splits * 8192 + g_force_row_tiles * 2;
#endif
    for (int i = 0; i < KEPT; ++i) {
        const int at = (last + i) % KEPT;
        if (std::memcmp(key, kept[at].key, sizeof key) == 0) {
            last = at;
            return kept[at].choice;
        }
    }
    last = oldest;
    oldest = (oldest + 1) % KEPT;
    kept[last].choice = make_choice(B, K_max, Hq, Hkv, D, max_pages, dtype);
    std::memcpy(kept[last].key, key, sizeof key);
    return kept[last].choice;
}

static bool attn_shape_ok(int32_t B, int32_t K_max, int32_t Hq, int32_t Hkv, int32_t D, int32_t max_pages) {
    return B >= 1 && B <= 65535 && K_max >= 1 && K_max <= GRAFT_MAX_NODES && Hq >= 1 && Hkv >= 1 &&
           Hkv <= 65535 && Hq % Hkv == 0 && Hq / Hkv <= 16 && (D == 64 || D == 128) && max_pages >= 1 &&
           max_pages <= AT_MAX_SPLITS * AT_MAX_SPLIT_PAGES;    // 64 splits x 4096 pages = 4 Mi tokens
}

thread_local ProfileHook g_prof;
#ifdef GRAFT_ATTN_STAMPS
static thread_local unsigned long long* g_stamps = nullptr;      // device buffer of the timing build
static thread_local size_t g_stamps_bytes = 0;
#endif

}  // namespace graft

extern "C" size_t graft_tree_attn_workspace_bytes(int32_t B, int32_t K_max, int32_t Hq, int32_t Hkv,
                                                  int32_t D, int32_t max_pages, int32_t dtype) {
    if (!graft::attn_shape_ok(B, K_max, Hq, Hkv, D, max_pages)) return 0;
    if (dtype != GRAFT_F32 && dtype != GRAFT_BF16) return 0;
    const graft::PathChoice& c = graft::choose_path(B, K_max, Hq, Hkv, D, max_pages, dtype);
    return c.direct ? c.dir.ws_bytes : c.mfma.ws_bytes;
}

extern "C" int32_t graft_attn_profile_events(void** start_events, void** stop_events, int32_t n) {
    if (n < 0 || (n > 0 && (!start_events || !stop_events))) return GRAFT_ERR_NULL;
    graft::g_prof = {reinterpret_cast<hipEvent_t*>(start_events), reinterpret_cast<hipEvent_t*>(stop_events), n, 0};
    return GRAFT_OK;
}

#ifdef GRAFT_ATTN_STAMPS
namespace graft {
// Timing build only: what the matrix cores of this chip deliver on a plain stream of independent
// v_mfma_f32_16x16x32_bf16 with operands of a given distribution (the clock under such a load
// depends on what the operands hold).  Every wavefront loads eight operands (64 lanes x 16 bytes
// each, the same for all wavefronts) and runs iters rounds of eight MFMAs on eight accumulators;
// every wavefront records real-time and core-clock counters around its loop (the wavefronts of a
// SIMD do not share the matrix core evenly: the oldest one runs first).
__global__ __launch_bounds__(1024) void mfma_calibration_kernel(const uintx4* __restrict__ operands, float* __restrict__ sink,
                                                               int iters, unsigned long long* __restrict__ stamps) {
    const int lane = threadIdx.x & 63;
    bf16x8 a[4], b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        a[j] = __builtin_bit_cast(bf16x8, operands[j * 64 + lane]);
        b[j] = __builtin_bit_cast(bf16x8, operands[(4 + j) * 64 + lane]);
    }
    floatx4 acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    const unsigned long long r0 = __builtin_amdgcn_s_memrealtime(), c0 = __builtin_readcyclecounter();
    for (int i = 0; i < iters; ++i) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j & 3], b[(j >> 1) & 3], acc[j], 0, 0, 0);
    }
    const unsigned long long c1 = __builtin_readcyclecounter(), r1 = __builtin_amdgcn_s_memrealtime();
    float t = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) t += acc[j][0] + acc[j][1] + acc[j][2] + acc[j][3];
    sink[static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x] = t;
    if (lane == 0) {
        unsigned long long* st = stamps + 4 * (static_cast<size_t>(blockIdx.x) * (blockDim.x >> 6) + (threadIdx.x >> 6));
        st[0] = r0;
        st[1] = r1;
        st[2] = c1 - c0;
        st[3] = 1;
    }
}
}  // namespace graft

// operands: 8 x 64 x 16 bytes; sink: n_workgroups * threads floats; stamps: 4 values per wavefront
// (real-time counter before and after the loop, core-clock cycles of the loop, 1).  threads is 256
// (one wavefront per SIMD), 512, 768 or 1024 (four).  All device memory, all the caller's.
extern "C" int32_t graft_mfma_calibration(const void* operands, float* sink, unsigned long long* stamps,
                                          int32_t n_workgroups, int32_t threads, int32_t iters, void* stream) {
    if (!operands || !sink || !stamps) return GRAFT_ERR_NULL;
    if (n_workgroups < 1 || n_workgroups > (1 << 20) || (threads != 256 && threads != 512 && threads != 768 && threads != 1024) || iters < 1 || iters > (1 << 24))
        return GRAFT_ERR_SHAPE;
    hipLaunchKernelGGL(graft::mfma_calibration_kernel, dim3(n_workgroups), dim3(threads), 0, static_cast<hipStream_t>(stream),
                       static_cast<const graft::uintx4*>(operands), sink, iters, stamps);
    return graft::check_launch();
}

// Timing build only (not part of the library's interface): device buffer that the MFMA kernel of
// this host thread's following graft_tree_attn calls fills with AT_STAMPS 64-bit values per
// workgroup; a call whose grid does not fit the buffer records nothing.  Null switches it off.
extern "C" int32_t graft_attn_stamp_buffer(void* device_buffer, size_t bytes) {
    graft::g_stamps = static_cast<unsigned long long*>(device_buffer);
    graft::g_stamps_bytes = device_buffer ? bytes : 0;
    return GRAFT_OK;
}
extern "C" int32_t graft_attn_stamp_count(void) { return graft::AT_STAMPS; }
// What a call of this shape launches: {1 for the MFMA path, 0 for the direct one; row blocks per wavefront; row tiles; splits}.
extern "C" int32_t graft_attn_plan(int32_t B, int32_t K_max, int32_t Hq, int32_t Hkv, int32_t D, int32_t max_pages, int32_t dtype,
                                   int32_t* plan) {
    if (!plan) return GRAFT_ERR_NULL;
    if (!graft::attn_shape_ok(B, K_max, Hq, Hkv, D, max_pages)) return GRAFT_ERR_SHAPE;
    const graft::PathChoice& c = graft::choose_path(B, K_max, Hq, Hkv, D, max_pages, dtype);
    plan[0] = c.direct ? 0 : 1;
    plan[1] = c.direct ? c.dir.mb : c.mfma.mb;
    plan[2] = c.direct ? c.dir.n_row_tiles : c.mfma.n_row_tiles;
    plan[3] = c.direct ? c.dir.n_splits : c.mfma.n_splits;
    return GRAFT_OK;
}
// The name of the call's main kernel, null where the shape is refused.
extern "C" const char* graft_attn_kernel_name(int32_t B, int32_t K_max, int32_t Hq, int32_t Hkv, int32_t D, int32_t max_pages, int32_t dtype) {
    if (!graft::attn_shape_ok(B, K_max, Hq, Hkv, D, max_pages)) return nullptr;
    const graft::PathChoice& c = graft::choose_path(B, K_max, Hq, Hkv, D, max_pages, dtype);
    if (c.direct) return c.dir.parts ? "tree_attn_parts_kernel" : "tree_attn_direct_kernel";
    return c.mfma.wide ? (c.mfma.mb == 2 ? "tree_attn_wide_128_kernel" : "tree_attn_wide_kernel") : "tree_attn_mfma_kernel";
}
// Holds the launch plan of this host thread's following calls (workspace query included) at
// n_splits splits and n_row_tiles row tiles where the shape allows them; zeros give the plan
// back to the cost model.
extern "C" int32_t graft_attn_force_plan(int32_t n_splits, int32_t n_row_tiles) {
    graft::g_force_splits = n_splits;
    graft::g_force_row_tiles = n_row_tiles;
    return GRAFT_OK;
}
#endif

extern "C" int32_t graft_tree_attn(const void* q, const void* k_cache, const void* v_cache,
                                   int64_t page_stride, int64_t token_stride, int64_t head_stride,
                                   const int32_t* block_table, int32_t max_pages,
                                   const int32_t* prefix_len, const int32_t* n_nodes, const uint64_t* mask,
                                   int32_t B, int32_t K_max, int32_t Hq, int32_t Hkv, int32_t D,
                                   int32_t page_size, float scale, int32_t dtype, void* out,
                                   void* workspace, size_t workspace_bytes, void* stream) {
    using namespace graft;
    if (!q || !k_cache || !v_cache || !block_table || !prefix_len || !n_nodes || !mask || !out)
        return GRAFT_ERR_NULL;
    if (dtype != GRAFT_F32 && dtype != GRAFT_BF16) return GRAFT_ERR_DTYPE;
    if (!attn_shape_ok(B, K_max, Hq, Hkv, D, max_pages) || page_size != GRAFT_PAGE_SIZE ||
        page_stride < 1 || token_stride < D || token_stride >= (1 << 26) || head_stride < D || token_stride % 8 != 0 ||
        head_stride % 8 != 0 || page_stride % 8 != 0 || !(scale > 0.f) || !(scale < 1e30f))
        return GRAFT_ERR_SHAPE;
    AttnParams p{};
    p.q = q; p.k = k_cache; p.v = v_cache; p.out = out;
    p.block_table = block_table; p.prefix_len = prefix_len; p.n_nodes = n_nodes;
    p.mask = reinterpret_cast<const u64*>(mask);
    p.page_stride = page_stride; p.token_stride = token_stride; p.head_stride = head_stride;
    p.max_pages = max_pages; p.B = B; p.K_max = K_max; p.Hq = Hq; p.Hkv = Hkv; p.G = Hq / Hkv;
    p.R = K_max * p.G;
    p.g_magic = (65536 + p.G - 1) / p.G;
    p.scale_log2e = scale * 1.4426950408889634f;
    hipStream_t s = static_cast<hipStream_t>(stream);

    const PathChoice& choice = choose_path(B, K_max, Hq, Hkv, D, max_pages, dtype);
    const auto fits = [&](size_t need) { return need == 0 || (workspace && workspace_bytes >= need); };
    const bool either = dtype == GRAFT_BF16 && D == AT_D;
    // bf16 with D = 128 and a workspace too small for the direct plan: the MFMA path if its own plan needs no more
    if (choice.direct && (!either || choice.only_direct || fits(choice.dir.ws_bytes) || !fits(choice.mfma.ws_bytes))) {
        const bool enough = fits(choice.dir.ws_bytes);
        if (!enough && either) return GRAFT_ERR_WORKSPACE;
        // (the other shapes have always run without a workspace: a caller that brings none, or too
        // little, gets a launch that does not split the keys over workgroups)
        return launch_direct(enough ? choice.dir : choice.unsplit, p, D, dtype, workspace, s);
    }

    const AttnPlan& pl = choice.mfma;
    if (!fits(pl.ws_bytes)) return GRAFT_ERR_WORKSPACE;
    p.R_pad = pl.r_pad; p.n_splits = pl.n_splits; p.n_row_tiles = pl.n_row_tiles;
    p.ws_o = static_cast<unsigned short*>(workspace);
    p.ws_ml = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + pl.ws_o_bytes);
    const dim3 grid(xcd_grid(static_cast<int64_t>(B) * Hkv * pl.n_splits, pl.n_row_tiles));
#ifdef GRAFT_ATTN_STAMPS
    p.stamps = static_cast<size_t>(grid.x) * AT_STAMPS * sizeof(unsigned long long) <= g_stamps_bytes ? g_stamps : nullptr;
#endif
    int32_t rc;
    if (pl.wide) {
        rc = launch_wide(64 * pl.mb, p, s);
    } else {
        switch (pl.mb) {
            case 1: launch_attn(tree_attn_mfma_kernel<1>, grid, dim3(AT_THREADS), 0, s, p, 1, 1); break;
            case 2: launch_attn(tree_attn_mfma_kernel<2>, grid, dim3(AT_THREADS), 0, s, p, 1, 1); break;
            case 3: launch_attn(tree_attn_mfma_kernel<3>, grid, dim3(AT_THREADS), 0, s, p, 1, 1); break;
            default: launch_attn(tree_attn_mfma_kernel<5>, grid, dim3(AT_THREADS), 0, s, p, 1, 1); break;
        }
        rc = check_launch();
    }
    if (rc != GRAFT_OK || pl.n_splits == 1) return rc;
    // wpt wavefronts per tile pair (cb_u splits each); as many tile pairs per workgroup as
    // make the workgroups one round (or, capped, a few whole rounds) over the compute units
    const int64_t n_tiles = static_cast<int64_t>(B) * Hkv * (pl.r_pad / 16) * (AT_D / 32);
    if (n_tiles > (1 << 30)) return GRAFT_ERR_SHAPE;
    const int cb_u = pl.n_splits > 12 ? 16 : pl.n_splits > 8 ? 12 : (pl.n_splits > 4 ? 8 : (pl.n_splits > 2 ? 4 : 2));
    const int wpt = (pl.n_splits + cb_u - 1) / cb_u;                       // 1 .. 4
    const int64_t cus = device_compute_units();
    int64_t tpw = (n_tiles + cus - 1) / cus;                               // tile pairs per workgroup
    const int64_t tpw_max = CB_MAX_WAVES / wpt;
    tpw = tpw < 1 ? 1 : (tpw > tpw_max ? tpw_max : tpw);
    const dim3 cgrid(static_cast<unsigned>((n_tiles + tpw - 1) / tpw)), cblock(static_cast<unsigned>(64 * tpw * wpt));
    const Magic n_blk = magic_any(static_cast<uint32_t>(p.R_pad / (pl.wide ? 32 : 16)));
    const auto combine = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, cgrid, cblock, 0, s, p.ws_o, p.ws_ml, n_nodes, static_cast<int32_t>(n_tiles),
                           static_cast<int32_t>(wpt | tpw << 8 | (256 + wpt - 1) / wpt << 16 | n_blk.shift << 25), p.R, p.R_pad, p.n_splits,
                           n_blk.m, Hkv, p);
    };
    const auto merge = [&](auto wide_) {
        constexpr bool WIDE = decltype(wide_)::value;
        switch (cb_u) {
            case 2: combine(tree_attn_combine_kernel<2, WIDE>); break;
            case 4: combine(tree_attn_combine_kernel<4, WIDE>); break;
            case 8: combine(tree_attn_combine_kernel<8, WIDE>); break;
            case 12: combine(tree_attn_combine_kernel<12, WIDE>); break;
            default: combine(tree_attn_combine_kernel<16, WIDE>); break;
        }
    };
    if (pl.wide) merge(std::true_type{});
    else merge(std::false_type{});
    return check_launch();
}
