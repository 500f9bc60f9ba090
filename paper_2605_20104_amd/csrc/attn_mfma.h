// What the kernels of the MFMA path of graft_tree_attn share (tree_attn.hip, tree_attn_wide.hip): sizes, time stamps, set-up,
// transfers from memory to LDS, accumulators in hand-placed AccVGPRs.
#pragma once
#include <type_traits>

#include "attn_shared.h"

namespace graft {

constexpr int AT_THREADS = 256;
constexpr int AT_WAVES = 4;
constexpr int AT_STAGE = 64;        // tokens per LDS stage (4 pages)
constexpr int AT_SUB = 32;          // tokens per softmax step
constexpr int AT_D = 128;
constexpr int AT_ROW_BYTES = AT_D * 2;
constexpr int AT_MAX_SPLITS = 64;

// Timing build (-DGRAFT_ATTN_STAMPS, a library of its own: see build.py): the MFMA kernel
// records when each workgroup passed the points below and writes them to a buffer the caller
// registered with graft_attn_stamp_buffer().  Times are values of the 100 MHz real-time counter
// (the first absolute, the others relative to it), two entries are the core-clock counter at
// both ends of the stage loop, which gives the clock the loop ran at.  Without the flag the
// macros are empty and the kernel is unchanged.
constexpr int AT_STAMPS = 24;
enum AttnStamp {
    AT_TS_START = 0,          // first instruction of the workgroup (absolute)
    AT_TS_LENGTHS = 1,        // lengths known
    AT_TS_TABLE_REQ = 2,      // block-table entries requested
    AT_TS_ZEROED = 3,         // accumulators zeroed
    AT_TS_STAGE0_REQ = 4,     // transfers of stage 0 issued
    AT_TS_TABLE_LDS = 5,      // table, masks and queries in LDS
    AT_TS_Q_DONE = 6,         // queries converted
    AT_TS_LOOP = 7,           // stage loop entered
    AT_TS_STAGE0 = 8,         // first stage arrived
    AT_TS_LOOP_END = 9,       // stage loop left
    AT_TS_END = 10,           // results written
    AT_TS_CYCLES_LOOP = 11,   // core-clock counter at AT_TS_LOOP
    AT_TS_CYCLES_END = 12,    // core-clock counter at AT_TS_LOOP_END
    AT_TS_STAGES = 13,        // stages of this workgroup
    AT_TS_VALID = 14,         // 1
    AT_TS_WAIT_CYCLES = 15,   // core-clock cycles wavefront 0 waited for its transfers of a stage, summed
    AT_TS_BARRIER_CYCLES = 16,  // ... and at the stage barriers (reading the counter costs some 50 cycles itself)
};
#ifdef GRAFT_ATTN_STAMPS
#define GRAFT_STAMPS_BEGIN()                                \
    unsigned long long at_stamp[AT_STAMPS] = {};            \
    at_stamp[AT_TS_START] = __builtin_amdgcn_s_memrealtime()
#define GRAFT_STAMP(k) (at_stamp[k] = __builtin_amdgcn_s_memrealtime() - at_stamp[AT_TS_START])
#define GRAFT_STAMP_CYCLES(k) (at_stamp[k] = __builtin_readcyclecounter())
#define GRAFT_SPAN_BEGIN() const unsigned long long at_span0 = __builtin_readcyclecounter()
#define GRAFT_SPAN_SPLIT(k) const unsigned long long at_span1 = __builtin_readcyclecounter(); at_stamp[k] += at_span1 - at_span0
#define GRAFT_SPAN_END(k) (at_stamp[k] += __builtin_readcyclecounter() - at_span1)
#define GRAFT_STAMPS_WRITE(p, n_stages)                                                     \
    do {                                                                                    \
        GRAFT_STAMP(AT_TS_END);                                                             \
        at_stamp[AT_TS_STAGES] = static_cast<unsigned long long>(n_stages);                 \
        at_stamp[AT_TS_VALID] = 1;                                                          \
        if (threadIdx.x == 0 && (p).stamps)                                                 \
            for (int at_k = 0; at_k < AT_STAMPS; ++at_k)                                    \
                (p).stamps[static_cast<size_t>(blockIdx.x) * AT_STAMPS + at_k] = at_stamp[at_k]; \
    } while (0)
#else
#define GRAFT_STAMPS_BEGIN() ((void)0)
#define GRAFT_STAMP(k) ((void)0)
#define GRAFT_STAMP_CYCLES(k) ((void)0)
#define GRAFT_SPAN_BEGIN() ((void)0)
#define GRAFT_SPAN_SPLIT(k) ((void)0)
#define GRAFT_SPAN_END(k) ((void)0)
#define GRAFT_STAMPS_WRITE(p, n_stages) ((void)0)
#endif

// The kernel with 32-row blocks (tree_attn_wide.hip): tiles of 128, 192, 256 or 384 rows.
int32_t launch_wide(int32_t tile_rows, const AttnParams& p, hipStream_t s);
int32_t launch_wide_128(const AttnParams& p, hipStream_t s);

struct SplitRange { int st0, st1, P, n, total; };       // stages, prefix length, nodes, tokens
__device__ __forceinline__ SplitRange split_range(const AttnParams& p, int n_raw, int P_raw, int split, int n_splits, uint32_t splits_magic) {
    SplitRange sr;
    const int n = n_raw < 1 || n_raw > p.K_max ? 0 : n_raw, cap = p.max_pages * GRAFT_PAGE_SIZE;
    sr.n = n;
    sr.P = P_raw < 0 ? 0 : (P_raw > cap ? cap : P_raw);
    sr.total = n ? ((sr.P + n) < cap ? (sr.P + n) : cap) : 0;
    const int n_stages = (sr.total + AT_STAGE - 1) / AT_STAGE;
    const int spt = div31(n_stages + n_splits - 1, splits_magic);
    sr.st0 = split * spt;
    sr.st1 = (sr.st0 + spt) < n_stages ? (sr.st0 + spt) : n_stages;
    if (sr.st1 < sr.st0) sr.st1 = sr.st0;
    return sr;
}

constexpr int AT_MAX_SPLIT_PAGES = 4096;          // block-table entries of one split kept in LDS
constexpr int AT_NBUF = 4;                         // LDS stage buffers
constexpr int AT_STAGE_BYTES = 2 * AT_STAGE * AT_ROW_BYTES;   // K rows then V rows
constexpr int AT_LOADS_PER_STAGE = 8;              // global->LDS instructions per wavefront per stage

// Global -> LDS without passing through registers: each lane's 16 bytes land at
// (wavefront-uniform LDS base) + lane * 16, so the swizzled LDS layout is produced by
// choosing which global chunk each lane fetches.  One instruction moves 4 token rows (1 KB)
// of K or of V; 4 wavefronts x 4 x (K,V) = one 64-token stage.
//
// The transfer is issued through inline assembly on purpose: the kernel keeps several stages
// in flight and waits for them with explicit s_waitcnt vmcnt(N); transfers the compiler knows
// about make it drain the whole vector memory counter before every LDS read and barrier.
// The global address is (wavefront-uniform 64-bit base) + (32-bit byte offset of the lane).
__device__ __forceinline__ void load_global_to_lds_b128(const void* base, unsigned lane_off, unsigned lds_addr) {
    // LDS address of lane l = M0 + 16 * l (M0 write needs one wait state before its use).
    // M0 is a reserved register the compiler sets up itself right before each of its own uses.
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_addr), "v"(lane_off), "s"(base)
                 : "memory");
}

// The same through a buffer descriptor: zeros where it ends in front of a lane's 16 (or 4) bytes.
constexpr unsigned BUFFER_WORD3 = 0x00020000u;  // raw buffer, 32-bit elements
__device__ __forceinline__ void buffer_to_lds_b128(const uintx4& descriptor, unsigned lane_off, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(lds_addr), "v"(lane_off), "s"(descriptor)
                 : "memory");
}
__device__ __forceinline__ void buffer_to_lds_b32(const uintx4& descriptor, unsigned lane_off, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :
                 : "s"(lds_addr), "v"(lane_off), "s"(descriptor)
                 : "memory");
}
__device__ __forceinline__ void load_global_to_lds_b32(const void* gptr, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                 :
                 : "s"(lds_addr), "v"(gptr)
                 : "memory");
}

__device__ __forceinline__ unsigned lds_address(const void* p) {
    return static_cast<unsigned>(reinterpret_cast<size_t>(
        (const __attribute__((address_space(3))) unsigned char*)(p)));
}

// ---- set-up: a chain of dependent trips to memory, lengths -> page table -> first keys.  Lengths and the first pages come
// through the scalar cache; what does not depend on them (ancestor masks, queries) is on its way to LDS meanwhile, and no load
// whose completion the compiler waits for is in flight with the transfers, which its counts do not know.
// Bound by those trips: with lengths, table entries and queries as vector loads, which return in order, the first keys were
// requested only when all queries had arrived and were converted, us after a workgroup's start: 3.4 -> 1.5 with 48 rows a
// wavefront (8 sequences of 4K keys), 1.3 -> 1.0 with 16 (one of 2K).  A round of 32 layers with 2K keys 442.0 -> 430.8 us, one
// layer with 32K keys 66.7 -> 64.7.
typedef const int32_t __attribute__((address_space(4)))* scalar_ptr;
__device__ __forceinline__ int scalar_load(const int32_t* p, int i) { return reinterpret_cast<scalar_ptr>(reinterpret_cast<size_t>(p))[i]; }

// Ancestor masks of sequence b to LDS, as 32-bit words; nodes past K_max get zeros.
__device__ __forceinline__ void request_masks(const AttnParams& p, int b, unsigned* Ms, int tid, int wave) {
    static_assert(GRAFT_MAX_NODES * GRAFT_MASK_WORDS * 2 == 2 * AT_THREADS, "two mask words per thread");
    const u64 at = reinterpret_cast<u64>(p.mask) + static_cast<u64>(b) * p.K_max * (GRAFT_MASK_WORDS * 8);
    const uintx4 d = {static_cast<unsigned>(at), static_cast<unsigned>(at >> 32), static_cast<unsigned>(p.K_max) * (GRAFT_MASK_WORDS * 8), BUFFER_WORD3};
    const unsigned to = __builtin_amdgcn_readfirstlane(lds_address(Ms)) + 256 * wave;
    buffer_to_lds_b32(d, 4 * tid, to);
    buffer_to_lds_b32(d, 4 * tid + 4 * AT_THREADS, to + 4 * AT_THREADS);
}
// The tile's queries to LDS, in the layout of K (16-byte chunk c of row r at c ^ (r & 15)); rows past the last one are zeros.
// Whole rows side by side: in operand layout, where a lane's 16 bytes lie in a row of their own, the requests of 192 rows held
// the compute unit's address path for more than a microsecond in front of everything else.
template <int TILE_ROWS>
__device__ __forceinline__ void request_queries(const AttnParams& p, int b, int g, int r_tile, unsigned lds, int lane, int wave) {
    const int l16 = lane & 15, lg = lane >> 4;
    const unsigned head = static_cast<unsigned>(g * p.G) * AT_ROW_BYTES;
    const u64 at = reinterpret_cast<u64>(p.q) + static_cast<u64>(b) * p.K_max * p.Hq * AT_ROW_BYTES + head;
    const uintx4 d = {static_cast<unsigned>(at), static_cast<unsigned>(at >> 32), static_cast<unsigned>(p.K_max * p.Hq) * AT_ROW_BYTES - head, BUFFER_WORD3};
#pragma unroll
    for (int j = 0; j < TILE_ROWS / 16; ++j) {
        const int rr = wave * (TILE_ROWS / 4) + 4 * j + lg, r = r_tile + rr;
        const int i = (r * p.g_magic) >> 16, hl = r - i * p.G;             // i = r / G
        const unsigned off = static_cast<unsigned>(i * p.Hq + hl) * AT_ROW_BYTES + (l16 ^ (rr & 15)) * 16;
        buffer_to_lds_b128(d, r < p.R ? off : ~15u, lds + (wave * (TILE_ROWS / 4) + 4 * j) * AT_ROW_BYTES);
    }
}

// s_waitcnt vmcnt(N) only (expcnt / lgkmcnt fields left at "no wait")
#define GRAFT_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(0x0F70 | ((N) & 15) | (((N) >> 4) << 14))

// Workgroup barrier that orders LDS traffic only.  __syncthreads() would also drain the
// vector memory counter and with it the global->LDS transfers of the stages still in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

#define GRAFT_ACC_BLOCK_0 "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31", "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47"
#define GRAFT_ACC_BLOCK_1 "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63", "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79", "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95"
#define GRAFT_ACC_BLOCK_2 "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111", "a112", "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127", "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143"
#define GRAFT_ACC_BLOCK_3 "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157", "a158", "a159", "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170", "a171", "a172", "a173", "a174", "a175", "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191"
#define GRAFT_ACC_BLOCK_4 "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207", "a208", "a209", "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223", "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239"
#define GRAFT_ACC_BLOCK_5 "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255"

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}
#define GRAFT_CONST(name, ic) constexpr int name = decltype(ic)::value

template <int R> __device__ __forceinline__ void acc_set(float v) {
    asm volatile("v_accvgpr_write_b32 a[%0], %1" : : "n"(R), "v"(v));
}
template <int R> __device__ __forceinline__ void acc_set_bits(unsigned v) {
    asm volatile("v_accvgpr_write_b32 a[%0], %1" : : "n"(R), "v"(v));
}
template <int R> __device__ __forceinline__ float acc_get() {
    float v;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(v) : "n"(R));
    return v;
}
template <int R> __device__ __forceinline__ void acc_scale(float a) {
    float t;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]\n\ts_nop 1\n\tv_mul_f32 %0, %0, %2\n\ts_nop 1\n\tv_accvgpr_write_b32 a[%1], %0"
                 : "=&v"(t)
                 : "n"(R), "v"(a));
}
// A register holding a bit pattern the compiler cannot see through (so it is kept, not
// rematerialised in front of an MFMA that reads it).
__device__ __forceinline__ unsigned opaque_bits(unsigned v) {
    unsigned r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "s"(v));
    return r;
}
#define GRAFT_MFMA_SETTLE() asm volatile("s_nop 15\n\ts_nop 7" ::: "memory")
// An empty asm that reads x: the registers of x stay allocated up to this point.  Used in the
// slow path after a group of MFMAs so that their source registers are not reused in between.
// (Not inside the pipeline regions: a use of an operand buffer after its reload has been
// issued makes the compiler wait for that reload, which undoes the prefetch.)
#define GRAFT_KEEP(x) asm volatile("" : : "v"(x))

// Rounds q * f to bf16 for two packed bf16 values.
__device__ __forceinline__ unsigned scale_bf16_pair(unsigned q2, float f) {
    return pack_bf16(__uint_as_float(q2 << 16) * f, __uint_as_float(q2 & 0xffff0000u) * f);
}
}  // namespace graft
