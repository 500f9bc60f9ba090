// graft_matrix_retrieve and graft_matrix_update: the transition matrix M[V][k] of successor
// ids that the method keeps in GPU memory.
//
// Retrieval is a gather along a static template: one 128-thread workgroup per sequence, one
// thread per template node.  A node's token is reached from the root's by as many dependent lookups in M as the node is
// deep, and the call is bound by those trips (nine for the paper's templates).  Every thread makes them for itself: it
// walks up the template once, with the ranks it passes as four bits each, and then down from the root; nodes
// that share ancestors read the same addresses.  (In rounds, one per depth, with two barriers of the workgroup each
// and the template requested behind the lengths: 2.5 us more a call for the nine levels, of about 6.)
//
// The refresh ranks every verified node's logits row.  Like the argmax of the acceptance
// step it is one HBM scan of the logits (4 V bytes per node): up to GRAFT_ARGMAX_CHUNKS workgroups
// per row; a workgroup finds a threshold from its threads' maxima, collects the few elements
// above it and picks its chunk's k best from those.  A key packs (logit,
// id) into 64 bits so that "larger logit first, then smaller id" is one unsigned compare.
// A one-wavefront kernel per node then merges the chunks, writes the greedy token and, if
// no later node carries the same token, the matrix row.  Few short rows go to one workgroup each, which does all of it.
// The threshold and the ranking of the few are one count of larger ones per lane each (kth_of, best_of) where k rounds of a wavefront
// maximum stood.  us a call in a graph, before / now: 1 x 40 rows of 128256 13.5 / 11.3, 8 x 24 of 32000 14.2 / 8.7, 8 x 128 of 32000
// 32.5 / 29.4, 4 x 64 of 65536 with k = 16 27.1 / 21.3, 16 x 16 of 8000 with k = 4 9.0 / 5.9.
#include <type_traits>

#include "common.h"

namespace graft {

constexpr int MR_THREADS = GRAFT_MAX_NODES;
constexpr int MU_THREADS = 256;
constexpr int MU_WAVES = MU_THREADS / 64;
constexpr int MM_UNROLL = 8;

__global__ __launch_bounds__(MR_THREADS) void matrix_retrieve_kernel(
    int32_t* __restrict__ n_nodes, const int32_t* __restrict__ n_ret, int32_t* __restrict__ tokens, int32_t K_max, int32_t N,
    const int32_t* __restrict__ tpl_parent, const int32_t* __restrict__ tpl_rank, const int32_t* __restrict__ M, int32_t V, int32_t k,
    int32_t* __restrict__ parent, int32_t* __restrict__ status) {
    const int b = blockIdx.x, u = threadIdx.x;
    __shared__ int32_t node[GRAFT_MAX_NODES];     // (template parent + 1) << 4 | rank
    __shared__ int32_t or_bad[2];
    static_assert(GRAFT_MAX_SUCCESSORS <= 16 && GRAFT_MAX_NODES == 128, "ranks in four bits, two wavefronts");
    int32_t* tok = tokens + static_cast<size_t>(b) * K_max;
    int32_t* par = parent + static_cast<size_t>(b) * K_max;
    const int32_t nd = n_nodes[b], nr = n_ret[b], root = tok[0];
    const int32_t f = u < N ? tpl_parent[u] : -1;
    const int32_t r = u < N ? tpl_rank[u] : 0;
    if (nd < 1 || nr < 0 || nr > N || nd + nr > K_max) {       // uniform over the workgroup
        if (u == 0) status[b] = GRAFT_STATUS_BAD_LENGTH;
        return;
    }
    const bool mine = u < nr;
    node[u] = mine ? ((f + 1) << 4) | (r & 15) : 0;
    if (workgroup_or_128(mine && (f < -1 || f >= u || r < 0 || r >= k), or_bad)) {
        if (u == 0) status[b] = GRAFT_STATUS_BAD_TREE;
        return;
    }
    if (mine) {
        // the walk up: the last sixteen ranks shifted in are those nearest the root, which come first on the way down
        u64 ranks = 0;
        int32_t depth = 0;
        for (int32_t j = u; j >= 0; ++depth) {
            const int32_t e = node[j];
            ranks = (ranks << 4) | static_cast<u64>(e & 15);
            j = (e >> 4) - 1;
        }
        int32_t t = root;
        for (int32_t at = 0;;) {
            const int32_t end = depth < at + 16 ? depth : at + 16;
            for (; at < end; ++at) {
                t = (t >= 0 && t < V) ? M[static_cast<size_t>(t) * k + static_cast<int32_t>(ranks & 15)] : -1;
                ranks >>= 4;
            }
            if (at >= depth) break;
            ranks = 0;                              // a deeper node: up again, as far as the next sixteen
            int32_t j = u;
            for (int32_t left = depth - at; left > 0; --left) {
                const int32_t e = node[j];
                ranks = (ranks << 4) | static_cast<u64>(e & 15);
                j = (e >> 4) - 1;
            }
        }
        tok[nd + u] = t;
        par[nd + u] = f < 0 ? 0 : nd + f;
    }
    if (u == 0) {
        n_nodes[b] = nd + nr;
        status[b] = 0;
    }
}

// ---- refresh ------------------------------------------------------------------------------

// (logit, id) -> key: larger logit = larger key; among equal logits the smaller id is larger.
__device__ __forceinline__ u64 rank_key(float v, int32_t id) {
    v += 0.0f;                                      // -0.0 -> +0.0: they compare equal
    const unsigned bits = __float_as_uint(v);
    const unsigned ord = (bits & 0x80000000u) ? ~bits : (bits | 0x80000000u);
    return (static_cast<u64>(ord) << 32) | static_cast<u64>(0xffffffffu - static_cast<unsigned>(id));
}
__device__ __forceinline__ int32_t key_id(u64 key) {
    return static_cast<int32_t>(0xffffffffu - static_cast<unsigned>(key & 0xffffffffu));
}

// The thread's KK best keys, best first.  Almost every element fails the first test (one
// float compare against the value of the worst kept key; equal values go on to the exact
// 64-bit compare because the id decides then).
template <int KK>
__device__ __forceinline__ void topk_insert(u64 (&top)[KK], float& worst, float v, int32_t id) {
    if (v >= worst) {
        u64 key = rank_key(v, id);
        if (key > top[KK - 1]) {
#pragma unroll
            for (int j = 0; j < KK; ++j) {
                if (key > top[j]) { const u64 t = top[j]; top[j] = key; key = t; }
            }
            // value of the new worst key (-inf while fewer than KK have been seen)
            const unsigned ord = static_cast<unsigned>(top[KK - 1] >> 32);
            const unsigned bits = (ord & 0x80000000u) ? (ord & 0x7fffffffu) : ~ord;
            worst = top[KK - 1] == 0 ? -INFINITY : __uint_as_float(bits);
        }
    }
}

// The scan of one thread's share of a chunk: take(value, id) for every element.
template <int THREADS, class Take>
__device__ __forceinline__ void scan_chunk(const float* __restrict__ row, const RowChunk& c, int tid, Take&& take) {
    if (tid < c.edge) take(row[c.edge_at(tid)], c.edge_at(tid));
    constexpr int U = 4;                            // 16-byte loads in flight per thread
    for (int32_t qd = c.q0 + tid; qd < c.q1; qd += U * THREADS) {
        float4 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t qu = qd + u * THREADS;
            x[u] = c.quad[qu < c.q1 ? qu : qd];     // a lane past the end re-reads its first quad (skipped below)
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t qu = qd + u * THREADS;
            if (qu < c.q1) {
                const int32_t e = c.head + qu * 4;
                take(x[u].x, e);
                take(x[u].y, e + 1);
                take(x[u].z, e + 2);
                take(x[u].w, e + 3);
            }
        }
    }
}

// k rounds over the workgroup: every wavefront offers its best remaining key, the owner of
// the round's winner (keys are unique: the id is part of them) pops it.
template <int KK, int WAVES>
__device__ __forceinline__ void select_rounds(u64 (&top)[KK], int k, u64 (&red)[2][WAVES], u64* out,
                                              int tid, int lane, int wave) {
    for (int j = 0; j < k; ++j) {
        const u64 wmax = wave_max_u64(top[0]);
        if (lane == 0) red[j & 1][wave] = wmax;
        __syncthreads();
        u64 gmax = red[j & 1][0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) gmax = red[j & 1][w] > gmax ? red[j & 1][w] : gmax;
        if (tid == 0) out[j] = gmax;
        if (gmax != 0 && top[0] == gmax) {
#pragma unroll
            for (int t = 0; t + 1 < KK; ++t) top[t] = top[t + 1];
            top[KK - 1] = 0;
        }
    }
}

// Maximum over 8 or 16 neighbouring lanes, all of them get it.
template <int N> __device__ __forceinline__ float lanes_max(float v) {
    static_assert(N == 8 || N == 16, "groups of a DPP row");
    v = __builtin_fmaxf(v, dpp_f32<0xB1>(v));
    v = __builtin_fmaxf(v, dpp_f32<0x4E>(v));
    v = __builtin_fmaxf(v, dpp_f32<0x141>(v));
    return N == 8 ? v : __builtin_fmaxf(v, dpp_f32<0x140>(v));
}
// The k-th largest of N maxima of disjoint groups of elements (in LDS): at least k elements are no smaller.  A lane counts what is larger
// than its own one; the smallest of those with fewer than k above them is the k-th.  (k rounds of a wavefront maximum, on which this
// stood before, took 8 to 16 times a chain of six dependent lane exchanges.)
template <int N> __device__ __forceinline__ float kth_of(const float* maxima, int k, int lane) {
    static_assert(N >= GRAFT_MAX_SUCCESSORS && N <= 64 && N % 4 == 0, "one a lane, k of them");
    const float own = maxima[lane % N];
    int above = 0;
#pragma unroll 1
    for (int t = 0; t < N / 4; ++t) {
        const float4 x = reinterpret_cast<const float4*>(maxima)[t];
        above += (x.x > own) + (x.y > own) + (x.z > own) + (x.w > own);
    }
    return -wave_max_f32(above < k ? -own : -INFINITY);
}
// The k best of n <= 256 keys in LDS by one wavefront, best first, 0 (no key) where there are fewer; put(j, key) by one lane each.
// Keys are unique, so a key's place is the number of larger ones, which every lane counts for its own where one a lane is enough.
template <class Put> __device__ __forceinline__ void best_of(const u64* keys, int n, int k, int lane, Put&& put) {
    if (n <= 64) {                                  // uniform
        const u64 own = lane < n ? keys[lane] : 0;
        int above = 0;
        for (int t = 0; t < n; t += 8) {
            u64 x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = keys[t + u];          // (behind the last one: whatever is there, not counted)
#pragma unroll
            for (int u = 0; u < 8; ++u) above += (t + u < n && x[u] > own) ? 1 : 0;
        }
        if (own != 0 && above < k) put(above, own);
        if (lane >= __builtin_popcountll(__builtin_amdgcn_ballot_w64(own != 0)) && lane < k) put(lane, 0);
        return;
    }
    u64 c[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) c[t] = (lane + t * 64) < n ? keys[lane + t * 64] : 0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int t = 0; t + 1 < 4 - a; ++t)
            if (c[t + 1] > c[t]) { const u64 sw = c[t]; c[t] = c[t + 1]; c[t + 1] = sw; }
    for (int j = 0; j < k; ++j) {
        const u64 gmax = wave_max_key(c[0]);
        if (lane == 0) put(j, gmax);
        if (gmax != 0 && c[0] == gmax) { c[0] = c[1]; c[1] = c[2]; c[2] = c[3]; c[3] = 0; }
    }
}

// Chunk scan: workgroup (chunk, node, sequence) -> its chunk's k best keys, best first.
//
// Fast path (chunks that fit in registers, MU_REG_QUADS 16-byte loads per thread and at most one
// edge element, all issued before anything else):
//   1. every thread takes the maximum of its elements (one max3 per two elements);
//   2. T is the k-th largest of the maxima of 16 or 32 groups of threads: at least k elements are >= T, so every one
//      of the chunk's k best is >= T;
//   3. the elements >= T (normally a dozen or two) are appended to a list in LDS as keys;
//   4. one wavefront ranks the list.
// If the list overflows (long runs of equal values) or the chunk does not fit, the
// workgroup takes the exact streaming path: per-thread sorted lists of KK >= k keys.
constexpr int MU_REG_QUADS = 12;                    // covers V <= 196608
static_assert(MU_REG_QUADS * MU_THREADS >= ROW_QUADS, "a chunk of the cut fits the registers, for V <= 196608");
constexpr int MU_LIST = 256;                        // four candidates per lane of the last wavefront

template <int KK, bool ONCE>
__global__ __launch_bounds__(MU_THREADS) void topk_chunk_kernel(
    const float* __restrict__ logits, const int32_t* __restrict__ n_nodes, int32_t K_max, int32_t V,
    int32_t per, int32_t k, u64* __restrict__ partial) {
    const int chunks = gridDim.x;
    const int chunk = blockIdx.x, i = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    u64* out = partial + ((static_cast<size_t>(b) * K_max + i) * chunks + chunk) * k;
    const int32_t n = n_nodes[b];
    if (i >= n || n > K_max) {                      // padding node
        if (tid < k) out[tid] = 0;
        return;
    }
    const float* row = logits + (static_cast<size_t>(b) * K_max + i) * V;
    const RowChunk c = row_chunk(row, V, chunk, chunks, per);
    const int32_t q0 = c.q0, q1 = c.q1;
    __shared__ u64 red[2][MU_WAVES];
    __shared__ u64 list[MU_LIST];
    __shared__ int32_t list_n;

    bool exact = true;
    if (q1 - q0 <= MU_REG_QUADS * MU_THREADS) {                      // uniform over the workgroup
        float4 x[MU_REG_QUADS];
        const float xe = tid < c.edge ? row[c.edge_at(tid)] : -INFINITY;
#pragma unroll
        for (int u = 0; u < MU_REG_QUADS; ++u) {
            const int32_t qu = q0 + tid + u * MU_THREADS;
            x[u] = qu < q1 ? load_logits<ONCE>(c.quad + qu) : float4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        }
        if (tid == 0) list_n = 0;
        float m = -INFINITY;
#pragma unroll
        for (int u = 0; u < MU_REG_QUADS; ++u)
            m = __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf(m, x[u].x), __builtin_fmaxf(x[u].y, x[u].z)), x[u].w);
        m = __builtin_fmaxf(m, xe);                                  // (last: it was requested last)
        // T = the k-th largest maximum of 16 groups of threads, of 32 where k is above 8 (the smallest of 16 would let in 50 elements)
        constexpr int GROUP = KK > 8 ? 8 : 16;
        __shared__ __attribute__((aligned(16))) float tops[MU_THREADS / GROUP];
        const float top = lanes_max<GROUP>(m);
        if (lane % GROUP == 0) tops[tid / GROUP] = top;
        __syncthreads();                                             // also orders list_n = 0 before the appends
        const float T = kth_of<MU_THREADS / GROUP>(tops, k, lane);
        if (tid < c.edge && xe >= T) {
            const int slot = atomicAdd(&list_n, 1);
            if (slot < MU_LIST) list[slot] = rank_key(xe, c.edge_at(tid));
        }
#pragma unroll
        for (int u = 0; u < MU_REG_QUADS; ++u) {
            const int32_t qu = q0 + tid + u * MU_THREADS;
            if (qu < q1) {
                const float e[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (e[t] >= T) {
                        const int slot = atomicAdd(&list_n, 1);
                        if (slot < MU_LIST) list[slot] = rank_key(e[t], c.head + qu * 4 + t);
                    }
                }
            }
        }
        __syncthreads();
        const int32_t nl = list_n;
        if (nl <= MU_LIST) {                                         // uniform
            if (wave == 0) best_of(list, nl, k, lane, [&](int j, u64 key) { out[j] = key; });
            exact = false;
        }
        __syncthreads();
    }
    if (!exact) return;

    // exact streaming path: per-thread sorted lists of KK keys
    u64 top[KK];
#pragma unroll
    for (int j = 0; j < KK; ++j) top[j] = 0;
    float worst = -INFINITY;
    scan_chunk<MU_THREADS>(row, c, tid, [&](float v, int32_t id) { topk_insert<KK>(top, worst, v, id); });
    select_rounds(top, k, red, out, tid, lane, wave);
}

// One wavefront per node: merge the chunks' keys, write the greedy token and the matrix row.
__global__ __launch_bounds__(64) void matrix_update_merge_kernel(
    const int32_t* __restrict__ tokens, const int32_t* __restrict__ n_nodes, int32_t V, int32_t B,
    int32_t K_max, int32_t k, int32_t chunks, const u64* __restrict__ partial, int32_t* __restrict__ M,
    int32_t* __restrict__ target_ids) {
    const int node = blockIdx.x;                    // b * K_max + i
    const int b = node / K_max, i = node - b * K_max;
    const int lane = threadIdx.x;
    const int32_t n = n_nodes[b];
    if (i >= n || n > K_max) {
        if (lane == 0) target_ids[node] = -1;
        return;
    }
    const u64* cand = partial + static_cast<size_t>(node) * chunks * k;
    const int n_cand = chunks * k;
    __shared__ u64 keys[GRAFT_ARGMAX_CHUNKS * GRAFT_MAX_SUCCESSORS];
    u64 c[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) c[t] = (lane + 64 * t) < n_cand ? cand[lane + 64 * t] : 0;
    // is this the last node (largest b, then i) carrying its token?
    const int32_t x = tokens[node];
    // The tokens of eight nodes per lane are requested at once, and only where one matches is the node looked at
    // (one node per lane and trip, its sequence's length with it: the merge of 2048 nodes took 13 us, 7 now)
    bool later = false;
    const int total = B * K_max;
    for (int o0 = node + 1; o0 < total && __builtin_amdgcn_ballot_w64(later) == 0; o0 += 64 * MM_UNROLL) {
        int32_t t[MM_UNROLL];
#pragma unroll
        for (int u = 0; u < MM_UNROLL; ++u) {
            const int o = o0 + lane + 64 * u;
            t[u] = tokens[o < total ? o : total - 1];
        }
#pragma unroll
        for (int u = 0; u < MM_UNROLL; ++u) {
            const int o = o0 + lane + 64 * u;
            if (t[u] == x && o < total) {
                const int ob = o / K_max, oi = o - ob * K_max;
                const int32_t on = n_nodes[ob];
                later = later || (oi < on && on <= K_max);
            }
        }
    }
    const bool write_row = x >= 0 && x < V && __builtin_amdgcn_ballot_w64(later) == 0;
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (lane + 64 * t < n_cand) keys[lane + 64 * t] = c[t];
    __syncthreads();                                // (one wavefront: LDS in order)
    best_of(keys, n_cand, k, lane, [&](int j, u64 key) {
        const int32_t id = key != 0 ? key_id(key) : -1;
        if (j == 0) target_ids[node] = id;
        if (write_row) M[static_cast<size_t>(x) * k + j] = id;
    });
}

// One launch for few rows that are short: a workgroup has a whole row, all of it on the way at once, ranks it as above and writes the
// greedy token and the matrix row itself.
constexpr int MW_THREADS = 1024;
constexpr int MW_QUADS = 8;                         // 16-byte loads in flight per thread: rows of up to MW_MAX elements
constexpr int32_t MW_MAX = 4 * MW_QUADS * MW_THREADS;
constexpr int64_t MW_ROWS = 256;

template <int KK>
__global__ __launch_bounds__(MW_THREADS) void topk_row_kernel(
    const int32_t* __restrict__ n_nodes, const int32_t* __restrict__ tokens, const float* __restrict__ logits, int32_t K_max, int32_t V,
    int32_t B, int32_t k, int32_t* __restrict__ M, int32_t* __restrict__ target_ids) {
    const int i = blockIdx.x, b = blockIdx.y, node = b * K_max + i;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t n = n_nodes[b];
    if (i >= n || n > K_max) {                      // padding node
        if (tid == 0) target_ids[node] = -1;
        return;
    }
    __shared__ u64 red[2][MW_THREADS / 64];
    __shared__ u64 list[MU_LIST];
    __shared__ u64 best[GRAFT_MAX_SUCCESSORS];
    __shared__ __attribute__((aligned(16))) float tops[MW_THREADS / 16];
    __shared__ int32_t list_n, later;
    const float* row = logits + static_cast<size_t>(node) * V;
    const RowChunk c = row_chunk(row, V, 0, 1, V / 4);
    const float xe = tid < c.edge ? row[c.edge_at(tid)] : -INFINITY;
    float4 x[MW_QUADS];
#pragma unroll
    for (int u = 0; u < MW_QUADS; ++u) {
        const int32_t qu = tid + u * MW_THREADS;
        x[u] = qu < c.q1 ? c.quad[qu] : float4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    }
    const int32_t t_own = tokens[node];
    if (tid == 0) list_n = later = 0;
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < MW_QUADS; ++u)
        m = __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf(m, x[u].x), __builtin_fmaxf(x[u].y, x[u].z)), x[u].w);
    m = __builtin_fmaxf(m, xe);
    const float top = lanes_max<16>(m);
    if ((lane & 15) == 0) tops[tid >> 4] = top;
    __syncthreads();                                // also orders list_n = later = 0 before what follows
    const float T = kth_of<MW_THREADS / 16>(tops, k, lane);
    const auto append = [&](float v, int32_t id) __attribute__((always_inline)) {
        if (v >= T) {
            const int slot = atomicAdd(&list_n, 1);
            if (slot < MU_LIST) list[slot] = rank_key(v, id);
        }
    };
    if (tid < c.edge) append(xe, c.edge_at(tid));
    if (m >= T) {                                   // (few threads)
#pragma unroll
        for (int u = 0; u < MW_QUADS; ++u) {
            const int32_t qu = tid + u * MW_THREADS, e = c.head + qu * 4;
            if (qu < c.q1) {
                append(x[u].x, e);
                append(x[u].y, e + 1);
                append(x[u].z, e + 2);
                append(x[u].w, e + 3);
            }
        }
    }
    // is this the last node (largest b, then i) carrying its token?
    for (int o = node + 1 + tid; o < B * K_max; o += MW_THREADS) {
        if (tokens[o] == t_own) {
            const int ob = o / K_max;
            const int32_t on = n_nodes[ob];
            if (o - ob * K_max < on && on <= K_max) later = 1;
        }
    }
    __syncthreads();
    const int32_t nl = list_n;
    if (nl <= MU_LIST) {
        if (wave > 0) return;
        best_of(list, nl, k, lane, [&](int j, u64 key) { best[j] = key; });
        wavefront_lds_order();
    } else {                                        // long runs of equal values: exact, per-thread sorted lists
        u64 own[KK];
#pragma unroll
        for (int j = 0; j < KK; ++j) own[j] = 0;
        float worst = -INFINITY;
        scan_chunk<MW_THREADS>(row, c, tid, [&](float v, int32_t id) { topk_insert<KK>(own, worst, v, id); });
        select_rounds(own, k, red, best, tid, lane, wave);
        __syncthreads();
        if (wave > 0) return;
    }
    if (lane < k) {
        const u64 key = best[lane];
        const int32_t id = key != 0 ? key_id(key) : -1;
        if (lane == 0) target_ids[node] = id;
        if (t_own >= 0 && t_own < V && later == 0) M[static_cast<size_t>(t_own) * k + lane] = id;
    }
}

}  // namespace graft

extern "C" int32_t graft_matrix_retrieve(const int32_t* M, int32_t V, int32_t k,
                                         const int32_t* tpl_parent, const int32_t* tpl_rank, int32_t N,
                                         const int32_t* n_ret, int32_t B, int32_t K_max,
                                         int32_t* tokens, int32_t* parent, int32_t* n_nodes, int32_t* status,
                                         void* stream) {
    if (!M || !tpl_parent || !tpl_rank || !n_ret || !tokens || !parent || !n_nodes || !status) return GRAFT_ERR_NULL;
    if (V < 1 || k < 1 || k > GRAFT_MAX_SUCCESSORS || N < 1 || N > GRAFT_MAX_NODES || B < 1 || K_max < 1 ||
        K_max > GRAFT_MAX_NODES)
        return GRAFT_ERR_SHAPE;
    hipLaunchKernelGGL(graft::matrix_retrieve_kernel, dim3(B), dim3(graft::MR_THREADS), 0,
                       static_cast<hipStream_t>(stream), n_nodes, n_ret, tokens, K_max, N, tpl_parent, tpl_rank, M, V, k,
                       parent, status);
    return graft::check_launch();
}

extern "C" size_t graft_matrix_update_workspace_bytes(int32_t B, int32_t K_max, int32_t V, int32_t k) {
    if (B < 1 || K_max < 1 || K_max > GRAFT_MAX_NODES || V < 1 || k < 1 || k > GRAFT_MAX_SUCCESSORS) return 0;
    return static_cast<size_t>(B) * K_max * GRAFT_ARGMAX_CHUNKS * k * sizeof(unsigned long long);
}

extern "C" int32_t graft_matrix_update(const int32_t* tokens, const int32_t* n_nodes, const float* logits,
                                       int32_t V, int32_t B, int32_t K_max, int32_t* M, int32_t k,
                                       int32_t* target_ids, void* workspace, size_t workspace_bytes,
                                       void* stream) {
    using namespace graft;
    if (!tokens || !n_nodes || !logits || !M || !target_ids) return GRAFT_ERR_NULL;
    if (B < 1 || B > 65535 || K_max < 1 || K_max > GRAFT_MAX_NODES || V < 1 || k < 1 ||
        k > GRAFT_MAX_SUCCESSORS || k > V || static_cast<int64_t>(B) * K_max > 65536)
        return GRAFT_ERR_SHAPE;
    const size_t need = graft_matrix_update_workspace_bytes(B, K_max, V, k);
    if (!workspace || workspace_bytes < need || (reinterpret_cast<size_t>(workspace) & 7) != 0)
        return GRAFT_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    u64* partial = static_cast<u64*>(workspace);
    // A row a workgroup, or several and a merge launch.  us a call in a graph, two launches / one:
    //   1 x 40 rows of 32000 8.8 / 8.2, 4 x 48 of 32000 11.5 / 9.7, 4 x 64 of 32000 with k = 16 14.1 / 11.1, 1 x 40 of 8000 8.8 / 5.4;
    //   longer rows, in two or more batches of loads, 1 x 40 of 50257 9.4 / 11.3, of 128256 11.3 / 14.0 (a compute unit on its own draws
    //   60 GB/s from memory); more rows than compute units, 8 x 48 of 8000 9.4 / 10.7, 16 x 64 12.9 / 20.1.
    // The host's side of a call 6.1 / 3.4 us.
    if (static_cast<int64_t>(B) * K_max <= MW_ROWS && V <= MW_MAX) {
        const dim3 grid(K_max, B);
        if (k <= 4) hipLaunchKernelGGL(topk_row_kernel<4>, grid, dim3(MW_THREADS), 0, s, n_nodes, tokens, logits, K_max, V, B, k, M, target_ids);
        else if (k <= 8) hipLaunchKernelGGL(topk_row_kernel<8>, grid, dim3(MW_THREADS), 0, s, n_nodes, tokens, logits, K_max, V, B, k, M, target_ids);
        else hipLaunchKernelGGL(topk_row_kernel<16>, grid, dim3(MW_THREADS), 0, s, n_nodes, tokens, logits, K_max, V, B, k, M, target_ids);
        return check_launch();
    }
    const RowCut cut = row_cut(static_cast<int64_t>(B) * K_max, V);
    dim3 grid(cut.chunks, K_max, B);
    const auto scan = [&](auto once_) {
        constexpr bool ONCE = decltype(once_)::value;
        const auto kernel = k <= 4 ? topk_chunk_kernel<4, ONCE> : (k <= 8 ? topk_chunk_kernel<8, ONCE> : topk_chunk_kernel<16, ONCE>);
        hipLaunchKernelGGL(kernel, grid, dim3(MU_THREADS), 0, s, logits, n_nodes, K_max, V, cut.per, k, partial);
    };
    if (read_once(static_cast<int64_t>(B) * K_max, V)) scan(std::true_type{});
    else scan(std::false_type{});
    int32_t rc = check_launch();
    if (rc != GRAFT_OK) return rc;
    hipLaunchKernelGGL(matrix_update_merge_kernel, dim3(B * K_max), dim3(64), 0, s, tokens, n_nodes, V, B, K_max, k,
                       cut.chunks, partial, M, target_ids);
    return check_launch();
}
