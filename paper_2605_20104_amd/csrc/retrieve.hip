// graft_retrieve: suffix n-gram lookup over the context token buffer.
//
// One workgroup per sequence, of 256, 512 or 1024 threads by the length of the rows.  The buffer is at most a few hundred
// KB, so the call is latency-bound, not bandwidth-bound: what matters is one
// launch, few dependent memory round trips, and an exact total order on the hits.
//
//   1. the lengths are requested first and, by the size of the workgroup, the first 2048, 8192 or 32768 tokens right
//      behind them, before the lengths are back (every index below L_max is readable); a thread loads groups of four
//      consecutive tokens with 16-byte loads.  A context of up to that many tokens goes to LDS at once
//      (at most 128 KB of the compute unit's 160), and the query (last n_max tokens of context ++ tail,
//      reversed) is read from there, each wavefront into a copy of its own: one memory round trip and
//      two barriers before the ranking.
//      A longer one is scanned from the registers it is loaded into, four units of 8192 tokens in
//      flight, no barrier and no copy in LDS: what bounds it is the compute unit's load path, 64
//      bytes a cycle.  A wavefront that has candidates copies its tokens to a piece of LDS of its own and walks there.
//      (All contexts through LDS in chunks of 16384, two barriers each and at most
//      one chunk in flight: 131072 tokens 14.1 us, 8.1 now; 40000 tokens 7.9, 6.6 now.)
//   2. scan: one compare per token against the query's last token, and a wavefront in which no
//      lane has it goes on (in text it is rare).  Otherwise the lanes test the token before as
//      well (in a register, or for the first of a group in LDS or from the lane below) where a hit
//      needs two tokens, and a candidate's match length is measured backwards, eight tokens per
//      round of independent reads;
//   3. a hit is the 64-bit key (match_len << 32 | e); each thread keeps its own best C keys in
//      registers (unrolled insertion, no dynamic indexing);
//   4. ranking without memory traffic.  The threads that have hits append their best C keys to a
//      short list in LDS (one 64-bit atomic reserves the places and counts the hits) and every
//      key counts how many of the list are larger: that is its rank (keys are unique because e
//      is).  A list that overflows (periodic text, tiny alphabets) takes the tournament instead:
//      each wavefront extracts its best C keys (exactly one lane owns a maximum and pops it),
//      wavefront 0 merges the C survivors of each (4, 8 or 16 of them) the same way.  C x m threads then copy the chains,
//      from LDS where the context is there.
//
// Measured on a 32768-token context (cycle stamps): with one position per lane and load, a
// dependent query load, a tournament in all 16 wavefronts it then had and a serial backward walk the kernel
// took 10.4 us; 2.3 us of that were the tournament (its vector instructions, issued by 16
// wavefronts that almost never hold a hit), 2 x 1.5 us the walks of the single wavefront per chunk
// that had a candidate (250 instructions of signed index arithmetic and per-token branches per
// round), 0.5 us each the dependent query load, the second chunk's barrier pair and the chain
// copy from memory.  That form took 6.1 us.  Since then, us a call in a graph: workgroups of four or eight wavefronts
// for rows of up to 8192 tokens, no branch around each group's load, and query copy and ranking per wavefront in place of
// two barriers, 2048 tokens 5.2 -> 3.7; all reads of a ranking round in flight (a condition in front of each had
// made them wait for one another), 4 x 8191 tokens of an alphabet of 20 12.2 -> 7.25.
#include "common.h"

namespace graft {

constexpr int RT_LIST = 128;                          // keys the ranking list holds before the tournament takes over
constexpr int RT_WALK = 8;                            // tokens compared per round of the backward match
constexpr int RT_FRONT = 32;                          // tokens in front of a position that a walk may read
static_assert(RT_FRONT % 4 == 0 && RT_FRONT <= 32 && RT_FRONT >= (GRAFT_MAX_NGRAM - 1 + RT_WALK - 1) / RT_WALK * RT_WALK, "whole rounds");
constexpr int RT_SLOTS = 4;                           // units of the streamed scan in flight
constexpr int RT_MOST = 1024;                         // threads of the largest workgroup, the one that streams
// Launch and barriers of a workgroup of sixteen wavefronts take longer than those of four, which shows where the tokens
// are few; but a thread compares its tokens one after the other, which shows where many of them are candidates.  So: the
// smallest workgroup whose one chunk holds the rows, by L_max, with two groups of four tokens per thread for the smallest
// (rows of 2048) and four for the others; the largest holds two chunks.  us a call, 256 / 512 / 1024 threads: 2048 tokens
// 3.7 / 4.0 / 4.4; 4096 tokens 3.84 / 3.77 / 4.7, of them equal, with n_max = 32, 23.6 / 17.5 / 20.5; 8192 tokens - / 4.0 / 4.9.
constexpr int rt_groups(int threads) { return threads == 256 ? 2 : 4; }     // groups of four consecutive tokens per thread and chunk
constexpr int rt_chunk(int threads) { return threads * 4 * rt_groups(threads); }     // tokens of a chunk
constexpr int rt_chunks(int threads) { return threads == RT_MOST ? 2 : 1; }
// Four consecutive tokens.  The context rows are only known to be 4-byte aligned (L_max is any
// number), which the hardware's vector loads accept.
struct __attribute__((packed, aligned(4))) Tok4 { int32_t t[4]; };

// The group of four tokens from i0 on, L_max >= 4: one 16-byte load per lane, consecutive lanes consecutive
// addresses.  The row's last group, if it is not whole, and those behind it are read from L_max - 4 on; shift_group
// then brings the tokens to their places (what lies past the row's end is arbitrary and never looked at).
__device__ __forceinline__ Tok4 load_group(const int32_t* __restrict__ x, int32_t i0, int32_t L_max) {
    return *reinterpret_cast<const Tok4*>(x + (i0 < L_max - 4 ? i0 : L_max - 4));
}
__device__ __forceinline__ void shift_group(Tok4& g, int32_t i0, int32_t L_max) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
        if (r < i0 - (L_max - 4)) { g.t[0] = g.t[1]; g.t[1] = g.t[2]; g.t[2] = g.t[3]; }
}

template <int RT_THREADS>
__global__ __launch_bounds__(RT_THREADS) void retrieve_kernel(
    const int32_t* __restrict__ ctx, const int32_t* __restrict__ ctx_len, int32_t L_max,
    const int32_t* __restrict__ tail, const int32_t* __restrict__ tail_len, int32_t tail_max,
    int32_t n_min, int32_t n_max, int32_t C, int32_t m,
    int32_t* __restrict__ chain_tok, int32_t* __restrict__ chain_len, int32_t* __restrict__ chain_pos,
    int32_t* __restrict__ chain_match, int32_t* __restrict__ n_hits, int32_t* __restrict__ status) {
    constexpr int RT_GROUPS = rt_groups(RT_THREADS), RT_WAVES = RT_THREADS / 64, RT_CHUNK = rt_chunk(RT_THREADS), RT_AHEAD = rt_chunks(RT_THREADS);
    constexpr int RT_UNIT = 8 * RT_THREADS;            // tokens of a unit of the streamed scan, two groups per thread
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the context, behind RT_FRONT slots that a walk reads where it passes the start (and ignores); a context that does not fit
    // is scanned in pieces of each wavefront's own
    __shared__ __attribute__((aligned(16))) int32_t front_and_ring[RT_FRONT + RT_AHEAD * RT_CHUNK];
    int32_t* const ring = front_and_ring + RT_FRONT;
    // the query from its end, one copy per wavefront (no barrier between writing and reading it); the backward match reads
    // up to RT_WALK entries past n_max - 1 and ignores them
    __shared__ int32_t queries[RT_WAVES][GRAFT_MAX_NGRAM + RT_WALK];
    __shared__ u64 red[RT_WAVES * GRAFT_MAX_CHAINS];   // per-wavefront best keys
    __shared__ u64 winners[RT_WAVES][GRAFT_MAX_CHAINS];   // the C winners, one copy per wavefront
    __shared__ __attribute__((aligned(16))) u64 list[RT_LIST];   // best keys of the threads that have hits, the rest zeros
    __shared__ u64 counts;                             // low word: keys appended to the list, high word: hits
    __shared__ int32_t tail_s[RT_THREADS];             // the first RT_THREADS tail tokens

    // the lengths first, the first chunks right behind them: they do not wait for the length, every
    // index below L_max is readable
    const int32_t L = ctx_len[b];
    const int32_t T = (tail != nullptr && tail_len != nullptr) ? tail_len[b] : 0;
    const int32_t* x = ctx + static_cast<size_t>(b) * L_max;
    Tok4 v[RT_AHEAD][RT_GROUPS];
    if (L_max >= 4) {
#pragma unroll
        for (int k = 0; k < RT_AHEAD; ++k)
#pragma unroll
            for (int u = 0; u < RT_GROUPS; ++u)
                if (k * RT_CHUNK + u * RT_THREADS * 4 < L_max)   // uniform: nothing is requested past the row's end
                    v[k][u] = load_group(x, k * RT_CHUNK + (u * RT_THREADS + tid) * 4, L_max);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[0][0].t[j] = 4 * tid + j < L_max ? x[4 * tid + j] : 0;
    }
    const int32_t tail_tok = (tail != nullptr && tid < tail_max) ? tail[static_cast<size_t>(b) * tail_max + tid] : 0;
    if (tid == 0) counts = 0;
    if (tid < RT_LIST) list[tid] = 0;
    u64* win = winners[wave];
    if (lane < GRAFT_MAX_CHAINS) win[lane] = 0;

    const bool bad = L < 0 || L > L_max || T < 0 || T > tail_max;

    int32_t* tok_b = chain_tok + static_cast<size_t>(b) * C * m;
    if (bad) {                                   // uniform over the workgroup
        for (int i = tid; i < C * m; i += RT_THREADS) tok_b[i] = -1;
        if (tid < C) {
            chain_len[b * C + tid] = 0;
            chain_pos[b * C + tid] = -1;
            chain_match[b * C + tid] = 0;
        }
        if (tid == 0) { n_hits[b] = 0; status[b] = GRAFT_STATUS_BAD_LENGTH; }
        return;
    }
    const int32_t QL = L + T;
    const int32_t nq = n_max < QL ? n_max : QL, qi = QL - 1 - lane;
    static_assert(GRAFT_MAX_NGRAM <= 64, "one query token per lane");
    int32_t* q_rev = queries[wave];
    const bool streamed = RT_THREADS == RT_MOST && L > RT_AHEAD * RT_CHUNK;   // (then L_max is larger as well: no group was cut short)
    if (streamed && lane < nq) q_rev[lane] = qi < L ? x[qi] : tail[static_cast<size_t>(b) * tail_max + (qi - L)];
    // Both chunks go to LDS at once (the token at position p sits at flat index p), and so do the tail tokens; the
    // query is then read from there: no second trip to memory.
    if (!streamed) {
#pragma unroll
        for (int k = 0; k < RT_AHEAD; ++k)
#pragma unroll
            for (int u = 0; u < RT_GROUPS; ++u) {
                const int32_t row0 = k * RT_CHUNK + u * RT_THREADS * 4;
                if (row0 >= L_max) continue;                     // uniform
                if ((L_max & 3) != 0 && L_max >= 4 && row0 + 4 * RT_THREADS > L_max) shift_group(v[k][u], row0 + 4 * tid, L_max);   // uniform
                *reinterpret_cast<int4*>(ring + row0 + tid * 4) = int4{v[k][u].t[0], v[k][u].t[1], v[k][u].t[2], v[k][u].t[3]};
            }
    }
    tail_s[tid] = tail_tok;
    __syncthreads();
    if (!streamed && lane < nq)
        q_rev[lane] = qi < L ? ring[qi] : ((qi - L) < RT_THREADS ? tail_s[qi - L] : tail[static_cast<size_t>(b) * tail_max + (qi - L)]);
    wavefront_lds_order();

    u64 top[GRAFT_MAX_CHAINS];
#pragma unroll
    for (int k = 0; k < GRAFT_MAX_CHAINS; ++k) top[k] = 0;
    int32_t my_hits = 0;

    // position i holds the token right before continuation start e = i + 1, 1 <= e <= L-1
    const int32_t last_i = L - 2;
    const int32_t n_chunks = last_i >= 0 ? last_i / RT_CHUNK + 1 : 0;
    const auto hit = [&](int32_t l, int32_t e) __attribute__((always_inline)) {
        ++my_hits;
        u64 key = (static_cast<u64>(l) << 32) | static_cast<u64>(e);
        // (only the best C of a thread can be among the best C overall)
#pragma unroll
        for (int kk = 0; kk < GRAFT_MAX_CHAINS; ++kk) {
            if (kk >= C) break;                   // uniform
            if (key > top[kk]) { const u64 u = top[kk]; top[kk] = key; key = u; }
        }
    };
    // How many tokens up to the one at `at` match the query's end, that one included, at most cap: RT_WALK are compared at
    // a time (independent LDS reads, those of the query's first round once for all candidates).
    int32_t q_first[RT_WALK];
#pragma unroll
    for (int jj = 0; jj < RT_WALK; ++jj) q_first[jj] = q_rev[1 + jj];
    const auto match_length = [&](const int32_t* at, int32_t cap) __attribute__((always_inline)) {
        int32_t l = 1, run = RT_WALK;             // run: matching tokens at the front of a round
        const auto compare = [&](int32_t base, const int32_t* q) __attribute__((always_inline)) {
            unsigned eq = 0;                      // bit jj: token base + jj before the last continues the match
#pragma unroll
            for (int jj = 0; jj < RT_WALK; ++jj) eq |= (at[-base - jj] == q[jj] && base + jj < cap) ? 1u << jj : 0u;
            run = __builtin_ctz(~eq);
            l += run;
        };
        if (cap > 1) compare(1, q_first);
        for (int32_t base = 1 + RT_WALK; run == RT_WALK && base < cap; base += RT_WALK) compare(base, q_rev + base);
        return l;
    };
    if (streamed) {
        // ---- a context that does not fit the ring: scanned from the registers it is loaded into
        const int32_t q_last = q_rev[0], q_prev = nq > 1 ? q_rev[1] : 0;
        const bool one = nq < 2 || n_max < 2;     // a query of one token
        constexpr int RT_PIECE = RT_FRONT + 256;  // tokens of a group row of one wavefront and those in front of it
        static_assert(RT_THREADS != RT_MOST || 2 * RT_WAVES * RT_PIECE <= RT_FRONT + RT_AHEAD * RT_CHUNK, "the pieces fit");
        int32_t* const piece = front_and_ring + wave * 2 * RT_PIECE;
        const auto scan = [&](Tok4 (&g)[2], int32_t unit) __attribute__((always_inline)) {
            unsigned cand = 0, longer = 0;        // bit 4 u + j: token j of group u is a candidate, the one before it matches too
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int32_t i0 = unit * RT_UNIT + (u * RT_THREADS + tid) * 4;
                const bool any = (g[u].t[0] == q_last) | (g[u].t[1] == q_last) | (g[u].t[2] == q_last) | (g[u].t[3] == q_last);
                if (__builtin_amdgcn_ballot_w64(any) == 0) continue;
                // the token before the group is the last of the lane below; lane 0 does not know it and lets the walk decide
                const int32_t below = __shfl_up(g[u].t[3], 1);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool more = !one && i0 + j >= 1 && (j == 0 ? lane == 0 || below == q_prev : g[u].t[j - 1] == q_prev);
                    if (i0 + j <= last_i && g[u].t[j] == q_last && (more || n_min < 2)) {
                        cand |= 1u << (4 * u + j);
                        longer |= more ? 1u << (4 * u + j) : 0u;
                    }
                }
            }
            if (__builtin_amdgcn_ballot_w64(cand != 0) == 0) return;
            // The walks read LDS: with a trip to memory for every candidate, a context that is nothing but candidates took
            // 2.6 times as long as with the context in LDS (131072 equal tokens, n_max = 32: 886 us, 285 like this; 335
            // through the ring in chunks).  The wavefront copies what it holds to its piece, and the tokens in front from
            // memory if a match can begin there.
            const u64 walks = __builtin_amdgcn_ballot_w64(longer != 0);
            if (walks != 0) {
                if ((walks & 0xff) != 0) {        // (those lanes' tokens are less than RT_FRONT from the piece's start)
                    const int32_t i = unit * RT_UNIT + ((lane >> 5) * RT_THREADS + wave * 64) * 4 - RT_FRONT + (lane & 31);
                    piece[(lane >> 5) * RT_PIECE + (lane & 31)] = x[i < 0 ? 0 : (i < L ? i : L - 1)];
                }
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    *reinterpret_cast<int4*>(piece + u * RT_PIECE + RT_FRONT + 4 * lane) = int4{g[u].t[0], g[u].t[1], g[u].t[2], g[u].t[3]};
                wavefront_lds_order();
            }
            while (cand != 0) {                   // one candidate per lane and pass
                const int bit = __builtin_ctz(cand);
                cand &= cand - 1;
                const int32_t e = unit * RT_UNIT + ((bit >> 2) * RT_THREADS + tid) * 4 + (bit & 3) + 1;
                const int32_t cap = (longer >> bit & 1) == 0 ? 1 : (n_max < e ? n_max : e);
                const int32_t l = match_length(piece + (bit >> 2) * RT_PIECE + RT_FRONT + 4 * lane + (bit & 3), cap);
                if (l >= n_min) hit(l, e);
            }
            wavefront_lds_order();                // (the next piece's writes stay behind these reads)
        };
        const int32_t n_units = last_i / RT_UNIT + 1;             // of 8192 tokens; the first RT_SLOTS are on their way
        Tok4 slot[RT_SLOTS][2], extra[RT_SLOTS - 1][2];
#pragma unroll
        for (int s = 0; s < RT_SLOTS; ++s)
#pragma unroll
            for (int u = 0; u < 2; ++u) slot[s][u] = v[s >> 1][2 * (s & 1) + u];
        const auto fetch = [&](Tok4 (&g)[2], int32_t unit) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 2; ++u) g[u] = load_group(x, unit * RT_UNIT + (u * RT_THREADS + tid) * 4, L_max);
        };
        const auto shift = [&](Tok4 (&g)[2], int32_t unit) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 2; ++u) shift_group(g[u], unit * RT_UNIT + (u * RT_THREADS + tid) * 4, L_max);
        };
        // No load in the loop is conditional: with a branch around it the compiler no longer knows how many are in
        // flight and waits for all of them.
        int32_t c = 0;
        for (; c + 2 * RT_SLOTS <= n_units; c += RT_SLOTS)
#pragma unroll
            for (int s = 0; s < RT_SLOTS; ++s) {
                scan(slot[s], c + s);
                fetch(slot[s], c + s + RT_SLOTS);
            }
        if (n_units > c + RT_SLOTS) {
#pragma unroll
            for (int s = 0; s < RT_SLOTS - 1; ++s) fetch(extra[s], c + s + RT_SLOTS);
        }
#pragma unroll
        for (int s = 0; s < RT_SLOTS; ++s) {
            shift(slot[s], c + s);
            scan(slot[s], c + s);
        }
#pragma unroll
        for (int s = 0; s < RT_SLOTS - 1; ++s)
            if (c + s + RT_SLOTS < n_units) {
                shift(extra[s], c + s + RT_SLOTS);
                scan(extra[s], c + s + RT_SLOTS);
            }
    } else {
#pragma unroll
        for (int c = 0; c < RT_AHEAD; ++c) {
            if (c >= n_chunks) continue;          // uniform over the workgroup (no break: c must stay a constant)
            const int32_t q_last = nq > 0 ? q_rev[0] : 0;
            // When a hit needs at least two matching tokens, the token before position i is
            // tested as well before the (divergent) walk: with frequent tokens at the end of
            // the query almost every wavefront would otherwise enter every walk.  Inside a
            // group that token is in a register; the one before the group comes from LDS.
            const bool two = n_min >= 2;
            const int32_t q_prev = nq > 1 ? q_rev[1] : 0;
            unsigned cand = 0;                    // bit 4 u + j: token j of group u is a candidate
#pragma unroll
            for (int u = 0; u < RT_GROUPS; ++u) {
                const int32_t i0 = c * RT_CHUNK + (u * RT_THREADS + tid) * 4;
                if (c * RT_CHUNK + u * RT_THREADS * 4 > last_i) continue;        // uniform: the whole group row is past the end
                // in text the query's last token is rare: one compare per token, and a wavefront in
                // which no lane has it skips the rest
                const bool any = (v[c][u].t[0] == q_last) | (v[c][u].t[1] == q_last) | (v[c][u].t[2] == q_last) |
                                 (v[c][u].t[3] == q_last);
                if (__builtin_amdgcn_ballot_w64(any) == 0) continue;
                const int32_t ip = i0 - 1;
                int32_t prev = ip >= 0 ? ring[ip] : ~q_prev;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int32_t t = v[c][u].t[j];
                    if (i0 + j <= last_i && t == q_last && (!two || (i0 + j >= 1 && prev == q_prev))) cand |= 1u << (4 * u + j);
                    prev = t;
                }
            }
            // one candidate per lane and pass (usually a single pass): the walk and the insertion
            // below exist once in the code and run once per pass, whatever slot the candidate is in
            while (cand != 0) {
                const int bit = __builtin_ctz(cand);
                cand &= cand - 1;
                const int32_t i = c * RT_CHUNK + ((bit >> 2) * RT_THREADS + tid) * 4 + (bit & 3);
                const int32_t e = i + 1;
                const int32_t l = match_length(ring + i, n_max < e ? n_max : e);
                if (l >= n_min) hit(l, e);
            }
        }
    }

    // ---- ranking.  Threads with hits append their best C keys (top[] is sorted, so its first
    //      min(my_hits, C) entries) to the list; the append order does not matter, a key's rank
    //      is the number of larger keys.
    if (my_hits > 0) {
        const int32_t k = my_hits < C ? my_hits : C;
        const u64 before = atomicAdd(&counts, (static_cast<u64>(my_hits) << 32) | static_cast<u64>(k));
        const int32_t off = static_cast<int32_t>(before & 0xffffffffu);
#pragma unroll
        for (int j = 0; j < GRAFT_MAX_CHAINS; ++j)
            if (j < k && off + j < RT_LIST) list[off + j] = top[j];
    }
    __syncthreads();
    const u64 counted = counts;
    const int32_t n_list = static_cast<int32_t>(counted & 0xffffffffu);
    if (wave * 64 >= C * m && wave > 0 && n_list <= RT_LIST) return;       // nothing to write for this wavefront
    if (n_list <= RT_LIST) {                      // uniform over the workgroup; every wavefront ranks for itself
        static_assert(RT_LIST == 128, "two keys per lane");
        const u64 k0 = list[lane], k1 = list[64 + lane];
        int32_t r0 = 0, r1 = 0;
        for (int32_t i0 = 0; i0 < n_list; i0 += 8) {              // eight keys per round, all reads in flight
            u64 kj[8];
#pragma unroll
            for (int u = 0; u < 8; u += 2) {
                const uint4 t = *reinterpret_cast<const uint4*>(&list[i0 + u]);
                kj[u] = (static_cast<u64>(t.y) << 32) | t.x;
                kj[u + 1] = (static_cast<u64>(t.w) << 32) | t.z;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                r0 += kj[u] > k0 ? 1 : 0;
                r1 += kj[u] > k1 ? 1 : 0;
            }
        }
        if (k0 != 0 && r0 < C) win[r0] = k0;
        if (k1 != 0 && r1 < C) win[r1] = k1;
        wavefront_lds_order();
    } else {
        // the list overflowed: every wavefront extracts its own best C keys (keys are unique because
        // e is, so exactly one lane owns each maximum and pops it), then wavefront 0 merges the
        // RT_WAVES x C survivors.  No memory access between the rounds.
        for (int c = 0; c < C; ++c) {
            const u64 wmax = wave_max_u64(top[0]);
            if (lane == 0) red[wave * GRAFT_MAX_CHAINS + c] = wmax;
            if (wmax != 0 && top[0] == wmax) {
#pragma unroll
                for (int k = 0; k + 1 < GRAFT_MAX_CHAINS; ++k) top[k] = top[k + 1];
                top[GRAFT_MAX_CHAINS - 1] = 0;
            }
        }
        __syncthreads();
        if (wave == 0) {
            // lane l holds candidates l and l + 64 of the RT_WAVES * C survivors (sorted pair)
            const int n_cand = RT_WAVES * C;
            u64 k0 = 0, k1 = 0;
            if (lane < n_cand) k0 = red[(lane / C) * GRAFT_MAX_CHAINS + lane % C];
            if (lane + 64 < n_cand) k1 = red[((lane + 64) / C) * GRAFT_MAX_CHAINS + (lane + 64) % C];
            if (k1 > k0) { const u64 t = k0; k0 = k1; k1 = t; }
            for (int c = 0; c < C; ++c) {
                const u64 gmax = wave_max_u64(k0);
                if (lane < RT_WAVES) winners[lane][c] = gmax;
                if (gmax != 0 && k0 == gmax) { k0 = k1; k1 = 0; }
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        n_hits[b] = static_cast<int32_t>(counted >> 32);
        status[b] = 0;
    }
    // ---- outputs: chain c starts at e = low word of win[c]; a context that fits LDS is still there
    if (tid < C) {
        const u64 key = win[tid];
        const int32_t e = static_cast<int32_t>(key & 0xffffffffu);
        const int32_t l = static_cast<int32_t>(key >> 32);
        const int32_t cl = key == 0 ? 0 : ((L - e) < m ? (L - e) : m);
        chain_pos[b * C + tid] = key == 0 ? -1 : e;
        chain_match[b * C + tid] = l;
        chain_len[b * C + tid] = cl;
    }
    for (int i = tid; i < C * m; i += RT_THREADS) {
        const int c = i / m, jj = i - c * m;
        const u64 key = win[c];
        const int32_t e = static_cast<int32_t>(key & 0xffffffffu);
        tok_b[i] = key == 0 || e + jj >= L ? -1 : (streamed ? x[e + jj] : ring[e + jj]);
    }
}

}  // namespace graft

extern "C" int32_t graft_retrieve(const int32_t* ctx, const int32_t* ctx_len, int32_t B, int32_t L_max,
                                  const int32_t* tail, const int32_t* tail_len, int32_t tail_max,
                                  int32_t n_min, int32_t n_max, int32_t C, int32_t m,
                                  int32_t* chain_tok, int32_t* chain_len, int32_t* chain_pos,
                                  int32_t* chain_match, int32_t* n_hits, int32_t* status, void* stream) {
    if (!ctx || !ctx_len || !chain_tok || !chain_len || !chain_pos || !chain_match || !n_hits || !status)
        return GRAFT_ERR_NULL;
    if ((tail == nullptr) != (tail_len == nullptr)) return GRAFT_ERR_NULL;
    if (B < 1 || L_max < 1 || L_max >= (1 << 30) || n_min < 1 || n_min > n_max ||
        n_max > GRAFT_MAX_NGRAM || C < 1 || C > GRAFT_MAX_CHAINS || m < 1 || m > (1 << 20) ||
        tail_max < 0 || (tail != nullptr && tail_max < 1))
        return GRAFT_ERR_SHAPE;
    const auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(B), dim3(threads), 0, static_cast<hipStream_t>(stream), ctx, ctx_len, L_max, tail, tail_len,
                           tail_max, n_min, n_max, C, m, chain_tok, chain_len, chain_pos, chain_match, n_hits, status);
    };
    if (L_max <= graft::rt_chunk(256)) launch(graft::retrieve_kernel<256>, 256);
    else if (L_max <= graft::rt_chunk(512)) launch(graft::retrieve_kernel<512>, 512);
    else launch(graft::retrieve_kernel<graft::RT_MOST>, graft::RT_MOST);
    return graft::check_launch();
}
