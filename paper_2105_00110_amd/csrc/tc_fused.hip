// Batched small graphs in one persistent launch.
//
// Every workgroup of k_fused_graphs pulls graph indices from a device
// counter and runs the whole path on one graph with workgroup-local steps, in
// one of three forms by the graph's size: everything in LDS (fused_small),
// per-vertex arrays in LDS (fused_medium), everything in the workspace
// (fused_large).  The steps, as the last one has them:
//
//   keys      each pair as lo * n + hi (lo < hi, ids local to the graph),
//             self-loops as the sentinel n * n;
//   sort      LSD radix sort of the keys, 8-bit digits, in the graph's
//             workspace (one digit histogram read for all passes; ranks by
//             8 ballots per key inside a wavefront, then wavefront offsets);
//   unique    distinct keys below the sentinel: the canonical edges
//             (u < v, lexicographic), m of them;
//   degree    d(v) by atomics on the canonical edges;
//   rank      sort of d(v) * n + v: the order (degree, id) of Sec.
//             "Notation", ties by smaller id; rank[v] and perm[r];
//   orient    each edge as rank(low) * n + rank(high) with its canonical
//             index as value, sorted: rows of N_H in rank space, ascending,
//             and their offsets;
//   count     one thread per oriented slot (r -> c) merges the tail of
//             N_H(r) after c with N_H(c), both sorted (the appendix's
//             Procedure 2 with counts in place of marks): every common w is
//             the triangle (r, c, w), found once from its lowest rank, and
//             adds 1 to the support of (r, w) and (c, w); the slot's own
//             support gains the number found;
//   tri       tri(v) = 1/2 Σ_{u ∈ N(v)} sup(v, u) and triG = 1/3 Σ_e sup(e)
//             (the quoted theorem of Sec. "Formulation");
//   aggregate num(v) = tri(v) + Σ_{u ∈ N(v)} (sup(v,u) > 0 ? 1 : 3) tri(u),
//             Definition 1's numerator times 3 with N△(v) read as the
//             neighbours sharing a triangle with v (Algorithm 2 in integer
//             form);
//   quotient  tc(v) = double(num) / double(3 triG), one IEEE division.
//
// Graphs of at most FUSED_MAX_N vertices qualify (keys stay below 2^32).
// Nothing is read back to the host and no memory is allocated, so the two
// launches can be captured in a graph and replayed.  tc_batch_fused takes
// its workspace from the caller; tc_batch_fused_noalloc uses a fixed device
// array of this file instead.
#include <mutex>

#include "tc_internal.h"
#include "tc_small.h"

namespace {

constexpr int64_t FUSED_MAX_N = 65535;
constexpr int FUSED_MW = 8;  // entries of each list per round of the count's merge
constexpr int FUSED_RB = 8;
constexpr int FUSED_RADIX = 1 << FUSED_RB;
constexpr int FUSED_ITEMS = 8;          // keys per thread in a scatter tile
constexpr int64_t FUSED_HEADER = 256;   // queue head and flags
// Workspace: a header, then 5 uint32 arrays per pair (the pair region,
// rounded up to 256 bytes), then per graph and vertex two uint64 and five
// uint32 arrays (40 bytes per vertex, 8 per graph for the extra row offset
// and alignment).
constexpr int64_t FUSED_PAIR_BYTES = 20;
constexpr int64_t FUSED_VTX_BYTES = 40;
constexpr int64_t FUSED_GRAPH_BYTES = 8;

__host__ __device__ inline int64_t pair_region(int64_t P) {
    return (FUSED_PAIR_BYTES * P + 255) / 256 * 256;
}

struct FusedArgs {
    const int32_t *src, *dst;
    const int64_t *pair_off, *vtx_off;
    const int32_t *order;
    int32_t G;
    int64_t P, N;
    int32_t *eu, *ev;
    uint64_t *sup;
    int64_t *num_edges;
    uint64_t *tri, *num;
    double *tc;
    uint64_t *triG;
    int32_t *status;
    unsigned char *ws;  // workspace (header first)
};

template <int BLOCK>
struct FusedLds {
    static constexpr int WAVES = BLOCK / TC_WAVE;
    uint32_t hist[4][FUSED_RADIX];  // digit counts of up to 4 passes, then running bases
    uint32_t wcnt[WAVES][FUSED_RADIX];
    uint32_t tot[FUSED_RADIX];
    uint32_t wsum[WAVES];
    uint64_t wsum64[WAVES];
};

// Atomic add ordered for the workgroup.  Every array these touch belongs to
// one graph and is read back only by the workgroup that owns it, after a
// barrier; device scope would make each fence write back and invalidate the
// L2, and the barriers' workgroup-scope release and acquire suffice.
template <typename T>
__device__ __forceinline__ void wg_add(T *p, T v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Sum of x over each run of equal keys among a wavefront's valid lanes, the
// keys non-decreasing in lane order: the run's last lane gets the run's sum
// and tail = true.
__device__ __forceinline__ uint64_t run_sum(uint32_t key, uint64_t x, bool valid, bool &tail) {
    const int lane = __lane_id();
    const uint32_t prev = __shfl_up(key, 1, TC_WAVE);
    const bool head = valid && (lane == 0 || prev != key);
    const uint64_t heads = __ballot(head);
    const uint64_t upto = heads & ((2ull << lane) - 1ull);  // heads at or below this lane
    const int start = upto ? 63 - __clzll(upto) : 0;
#pragma unroll
    for (int off = 1; off < TC_WAVE; off <<= 1) {
        const uint64_t y = __shfl_up(x, off, TC_WAVE);
        if (lane - off >= start) x += y;
    }
    const uint32_t next = __shfl_down(key, 1, TC_WAVE);
    const uint64_t live = __ballot(valid);
    const bool next_live = lane < TC_WAVE - 1 && ((live >> (lane + 1)) & 1ull);
    tail = valid && (!next_live || next != key);
    return x;
}

__device__ __forceinline__ int fused_bits(uint32_t max_value) {
    return max_value == 0 ? 0 : 32 - __clz(max_value);
}

// Sum over the workgroup (every thread returns it).
template <int BLOCK>
__device__ __forceinline__ uint64_t block_sum64(uint64_t x, FusedLds<BLOCK> &sh) {
    x = tc_wave_sum(x);
    if (__lane_id() == 0) sh.wsum64[threadIdx.x / TC_WAVE] = x;
    __syncthreads();
    uint64_t t = 0;
#pragma unroll
    for (int q = 0; q < FusedLds<BLOCK>::WAVES; ++q) t += sh.wsum64[q];
    __syncthreads();
    return t;
}

template <int BLOCK>
__device__ __forceinline__ uint32_t block_max32(uint32_t x, FusedLds<BLOCK> &sh) {
    x = tc_wave_max(x);
    if (__lane_id() == 0) sh.wsum[threadIdx.x / TC_WAVE] = x;
    __syncthreads();
    uint32_t t = 0;
#pragma unroll
    for (int q = 0; q < FusedLds<BLOCK>::WAVES; ++q) t = sh.wsum[q] > t ? sh.wsum[q] : t;
    __syncthreads();
    return t;
}

// Exclusive prefix of v[0..256) in place; threads below 256 hold one digit.
template <int BLOCK>
__device__ __forceinline__ void scan256(uint32_t *v, FusedLds<BLOCK> &sh) {
    static_assert(BLOCK >= FUSED_RADIX, "one digit per thread");
    const int tid = threadIdx.x;
    const uint32_t x = tid < FUSED_RADIX ? v[tid] : 0u;
    const uint32_t incl = tc_wave_incl_scan(x);
    if (tid < FUSED_RADIX && __lane_id() == TC_WAVE - 1) sh.wsum[tid / TC_WAVE] = incl;
    __syncthreads();
    if (tid < FUSED_RADIX) {
        uint32_t before = 0;
        for (int q = 0; q < tid / TC_WAVE; ++q) before += sh.wsum[q];
        v[tid] = before + incl - x;
    }
    __syncthreads();
}

// Stable LSD radix sort of n keys (and values) held in device memory, by
// the whole workgroup.  The sorted data ends in *k / *v; the other buffers
// are ping-pong space.  One read of the keys counts the digits of every
// pass (the multiset of keys is the same before each pass).
template <int BLOCK, bool VAL>
__device__ __forceinline__ void block_sort(uint32_t *&k, uint32_t *&kt, uint32_t *&v, uint32_t *&vt, uint32_t n,
                           int bits, FusedLds<BLOCK> &sh) {
    constexpr int WAVES = FusedLds<BLOCK>::WAVES;
    constexpr int TILE = BLOCK * FUSED_ITEMS;
    const int passes = (bits + FUSED_RB - 1) / FUSED_RB;
    if (n <= 1 || passes == 0) return;
    const int tid = threadIdx.x, w = tid / TC_WAVE, lane = __lane_id();
    const uint64_t lt = tc_lanemask_lt();
    for (int i = tid; i < 4 * FUSED_RADIX; i += BLOCK) (&sh.hist[0][0])[i] = 0;
    __syncthreads();
    for (uint32_t i = tid; i < n; i += BLOCK) {
        const uint32_t key = k[i];
        for (int p = 0; p < passes; ++p) atomicAdd(&sh.hist[p][(key >> (FUSED_RB * p)) & 255u], 1u);
    }
    __syncthreads();
    for (int p = 0; p < passes; ++p) scan256(sh.hist[p], sh);
    for (int p = 0; p < passes; ++p) {
        const int shift = FUSED_RB * p;
        uint32_t *base = sh.hist[p];
        for (uint32_t t0 = 0; t0 < n; t0 += TILE) {
            for (int i = tid; i < WAVES * FUSED_RADIX; i += BLOCK) (&sh.wcnt[0][0])[i] = 0;
            __syncthreads();
            uint32_t key[FUSED_ITEMS], val[FUSED_ITEMS], rnk[FUSED_ITEMS];
            const uint32_t wb = t0 + (uint32_t)w * (TC_WAVE * FUSED_ITEMS);
#pragma unroll
            for (int it = 0; it < FUSED_ITEMS; ++it) {
                const uint32_t i = wb + it * TC_WAVE + lane;
                const bool valid = i < n;
                key[it] = valid ? k[i] : 0u;
                if constexpr (VAL) val[it] = valid ? v[i] : 0u;
            }
            // rank among equal digits: earlier items of the wavefront, then
            // lower lanes of the same item (memory order)
#pragma unroll
            for (int it = 0; it < FUSED_ITEMS; ++it) {
                const uint32_t i = wb + it * TC_WAVE + lane;
                const bool valid = i < n;
                const uint32_t d = (key[it] >> shift) & 255u;
                uint64_t peers = __ballot(valid);
#pragma unroll
                for (int b = 0; b < FUSED_RB; ++b) {
                    const bool bit = (d >> b) & 1u;
                    const uint64_t bal = __ballot(bit);
                    peers &= bit ? bal : ~bal;
                }
                uint32_t prior = 0;
                if (valid) prior = sh.wcnt[w][d];
                rnk[it] = prior + (uint32_t)__popcll(peers & lt);
                // every lane has read the count before the highest peer
                // replaces it (a wavefront's LDS operations run in order)
                __builtin_amdgcn_wave_barrier();
                if (valid && (peers >> lane) == 1ull) sh.wcnt[w][d] = prior + (uint32_t)__popcll(peers);
            }
            __syncthreads();
            if (tid < FUSED_RADIX) {
                uint32_t run = 0;
                for (int q = 0; q < WAVES; ++q) {
                    const uint32_t c = sh.wcnt[q][tid];
                    sh.wcnt[q][tid] = run;
                    run += c;
                }
                sh.tot[tid] = run;
            }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < FUSED_ITEMS; ++it) {
                const uint32_t i = wb + it * TC_WAVE + lane;
                if (i < n) {
                    const uint32_t d = (key[it] >> shift) & 255u;
                    const uint32_t pos = base[d] + sh.wcnt[w][d] + rnk[it];
                    kt[pos] = key[it];
                    if constexpr (VAL) vt[pos] = val[it];
                }
            }
            __syncthreads();
            if (tid < FUSED_RADIX) base[tid] += sh.tot[tid];
            __syncthreads();
        }
        uint32_t *t = k;
        k = kt;
        kt = t;
        if constexpr (VAL) {
            t = v;
            v = vt;
            vt = t;
        }
    }
}

// The distinct keys of the sorted a[0..n) that lie below `limit`, in order,
// written to out; returns their count.
template <int BLOCK>
__device__ __forceinline__ uint32_t block_unique(const uint32_t *a, uint32_t n, uint32_t limit, uint32_t *out,
                                 FusedLds<BLOCK> &sh) {
    constexpr int WAVES = FusedLds<BLOCK>::WAVES;
    const int w = threadIdx.x / TC_WAVE;
    uint32_t count = 0;
    for (uint32_t t0 = 0; t0 < n; t0 += BLOCK) {
        const uint32_t i = t0 + threadIdx.x;
        bool keep = false;
        uint32_t key = 0;
        if (i < n) {
            key = a[i];
            keep = key < limit && (i == 0 || a[i - 1] != key);
        }
        const uint64_t bal = __ballot(keep);
        if (__lane_id() == 0) sh.wsum[w] = (uint32_t)__popcll(bal);
        __syncthreads();
        uint32_t before = 0, all = 0;
#pragma unroll
        for (int q = 0; q < WAVES; ++q) {
            const uint32_t c = sh.wsum[q];
            before += q < w ? c : 0u;
            all += c;
        }
        if (keep) out[count + before + (uint32_t)__popcll(bal & tc_lanemask_lt())] = key;
        count += all;
        __syncthreads();
    }
    return count;
}

// Writes the outputs of a graph that is not computed (status < 0): no
// edges, zero counts and quotients for its vertices.
template <int BLOCK>
__device__ __forceinline__ void fused_fail(const FusedArgs &a, int32_t g, int64_t va, int64_t n, int32_t st) {
    for (int64_t v = threadIdx.x; v < n; v += BLOCK) {
        if (a.tri) a.tri[va + v] = 0;
        if (a.num) a.num[va + v] = 0;
        if (a.tc) a.tc[va + v] = 0.0;
    }
    if (threadIdx.x == 0) {
        a.num_edges[g] = 0;
        if (a.triG) a.triG[g] = 0;
        a.status[g] = st;
    }
}

// Any thread's flag, as a scalar: branches on it stay uniform.
__device__ __forceinline__ bool wg_any(bool x) {
    return __builtin_amdgcn_readfirstlane(__syncthreads_or(x)) != 0;
}

// A graph of the batch: where its pairs and vertices lie, and its slice of the
// workspace (five uint32 arrays per pair, then the vertex arrays).
struct GraphRef {
    int32_t g;
    int64_t pa, va;
    uint32_t n, P;
    uint32_t *A, *B, *C, *D, *E;
    uint64_t *triR, *numR;
    uint32_t *deg, *rank, *perm, *vtmp, *orp;  // orp[n + 1]
};

// ---------------------------------------------------------------------------
// Graphs that fit LDS (at most 16 pairs per thread): tc_small.h's steps, the
// slot merge and the sums in LDS, outputs straight from registers.  Bound by
// LDS and VALU work between some forty barriers; in device memory the same
// steps were bound by the memory latency that 16 wavefronts cannot cover (five
// ER graphs of 10 k pairs at once: 237 us a call before, 90 us so).
// ---------------------------------------------------------------------------
template <int BLOCK>
__device__ __forceinline__ void fused_small(const FusedArgs &a, const GraphRef q, tc_small::Lds<BLOCK> &L) {
    using namespace tc_small;
    const uint32_t n = q.n, P = q.P;
    const int b = bits_of(n > 1 ? n - 1 : 1);
    const int itn = P == 0 ? 1 : (int)((P + BLOCK - 1) / BLOCK);
    const uint32_t none = (uint32_t)((1ull << (2 * b)) - 1ull);
    uint32_t key[ITEMS];
    bool bad = false;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        key[it] = none;
        if (it < itn) {
            const uint32_t i = elem(it, itn);
            if (i < P) {
                const uint32_t x = (uint32_t)a.src[q.pa + i], y = (uint32_t)a.dst[q.pa + i];
                if (x >= n || y >= n) bad = true;
                else if (x != y) key[it] = (x < y ? x << b | y : y << b | x);
            }
        }
    }
    if (wg_any(bad)) {
        fused_fail<BLOCK>(a, q.g, q.va, n, TC_ERR_VERTEX_RANGE);
        return;
    }
    Edges E;
    const uint32_t m = canonical<BLOCK>(key, itn, b, E, L);
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        if (E.ends[it] != NONE) {
            if (a.eu) a.eu[q.pa + E.tag[it]] = (int32_t)(E.ends[it] >> 16);
            if (a.ev) a.ev[q.pa + E.tag[it]] = (int32_t)(E.ends[it] & 0xFFFFu);
        }
    (void)degree_rank<BLOCK>(E, n, L, [](uint32_t, uint32_t) {});
    (void)orient<BLOCK>(E, n, m, L);
    count_slots<BLOCK>(m, n, L);
    if (a.sup) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            if (E.ends[it] != NONE)
                a.sup[q.pa + (E.tag[it] & 0xFFFFu)] = support(E.tag[it] >> 16, L);
    }
    const uint32_t three_t = slot_sums<BLOCK>(m, L);
    bool odd = three_t % 3 != 0;
    const uint32_t *const tri = L.tri, *const num = L.num;
    const uint64_t tg = three_t / 3;
    for (uint32_t v = threadIdx.x; v < n; v += BLOCK) {
        const uint32_t r = L.rank[v];
        odd |= (tri[r] & 1u) != 0;
        const uint64_t t = tri[r] >> 1, x = num[r] + t;
        if (a.tri) a.tri[q.va + v] = t;
        if (a.num) a.num[q.va + v] = x;
        if (a.tc) a.tc[q.va + v] = tg == 0 ? 0.0 : __ddiv_rn((double)x, (double)(3 * tg));
    }
    odd = wg_any(odd);
    if (threadIdx.x == 0) {
        a.num_edges[q.g] = m;
        if (a.triG) a.triG[q.g] = tg;
        a.status[q.g] = odd ? TC_ERR_DEVICE : (tg == 0 ? TC_TRIANGLE_FREE : TC_OK);
    }
}

// ---------------------------------------------------------------------------
// Graphs of up to 2^20 pairs whose per-vertex arrays fit LDS: the pairs and
// slots stay in the workspace, read and written in tiles of 8 or 16 elements a
// thread, all loads of a tile issued before the first use; every per-vertex
// count, offset, rank and sum that the edges gather or add to is in LDS.  Bound
// by the memory latency of one workgroup's 16 wavefronts, so loads in flight
// count: a loop over single elements waits a round trip for each (4096 BA
// graphs: 25.8 ms before, 14.9 ms so, of which the merge's random rows took 8.4;
// 10.65 ms with the highest rows and their counts in LDS, 10.1 with the supports
// of the others on their slots).
// ---------------------------------------------------------------------------
template <int BLOCK>
struct Medium {
    static constexpr uint32_t NMAX = 21 * BLOCK;
    static constexpr uint32_t PMAX = 1u << 20;
    static constexpr uint32_t LT = 8 * BLOCK;   // elements per tile of the loops
    static constexpr uint32_t ST = 16 * BLOCK;  // of the sort
    static constexpr uint32_t CT = 4 * BLOCK;   // of the merge (8: 10.71 ms, 2: 10.72)
    // longest oriented row: d+ neighbours of degree >= d+ each, so d+^2 <= 2m
    static constexpr uint32_t HALO = 1536;
    // bytes: per-vertex words and the row sort's tile with its halo, or a rank
    // and a cursor per vertex, or the sort's exchange and digit counts
    static constexpr size_t ROWS = 4 * (size_t)NMAX + 4 * (LT + 2 * HALO);
    static constexpr size_t ORIENT = 6 * (size_t)NMAX;
    static constexpr size_t SORT = 4 * (size_t)ST + 4 * (size_t)(BLOCK / TC_WAVE) * tc_small::RADIX;
    // what is left of a workgroup's share of LDS: the merge's cache
    static constexpr size_t COUNT = 150 * (size_t)BLOCK;
    static constexpr size_t max2(size_t x, size_t y) { return x > y ? x : y; }
    static constexpr size_t BYTES = max2(max2(ROWS, ORIENT), max2(SORT, COUNT));
    static constexpr uint32_t PAD = 8;  // a window of the merge past its row
    static_assert(BYTES / 4 - NMAX >= CT + HALO + PAD, "a tile of the merge fits after the row ends");
};

// Digit counts of up to 4 passes, running bases during a pass; scan words.
template <int BLOCK>
struct MediumTail {
    uint32_t hist[4][tc_small::RADIX];
    uint32_t wsum[BLOCK / TC_WAVE + 1];
};

// The arena of a workgroup, used by one tier at a time.
template <int BLOCK>
union FusedArena {
    tc_small::Lds<BLOCK> small;
    FusedLds<BLOCK> large;
    struct {
        unsigned char raw[Medium<BLOCK>::BYTES];
        MediumTail<BLOCK> tail;
    } medium;
};

// Passes and digit width of a sort on `bits` bits (at most 8 a pass).
struct SortPlan {
    int shift, bits, passes, width;
    __device__ SortPlan(int sh, int bt) : shift(sh), bits(bt) {
        passes = (bits + 7) / 8;
        width = (bits + passes - 1) / passes;
    }
    __device__ int at(int p) const { return shift + p * width; }
    __device__ int bits_at(int p) const {
        const int left = bits - p * width;
        return width < left ? width : left;
    }
};

template <int BLOCK>
__device__ __forceinline__ void medium_hist(const SortPlan &sp, uint32_t key, MediumTail<BLOCK> &T) {
#pragma unroll
    for (int p = 0; p < 4; ++p)
        if (p < sp.passes)
            atomicAdd(&T.hist[p][(key >> sp.at(p)) & ((1u << sp.bits_at(p)) - 1u)], 1u);
}

// Element i of a slice of under 2^32 bytes: a scalar base and a 32-bit offset
// (64-bit addresses for every load in flight cost the tiles their registers).
template <typename T>
__device__ __forceinline__ T &at(T *base, uint32_t i) {
    return *reinterpret_cast<T *>(reinterpret_cast<uintptr_t>(base) + (uintptr_t)(i * (uint32_t)sizeof(T)));
}

// Stable sort of k[0..n) (result in k, kt the other buffer) with the digit
// counts of every pass already in T.hist.
template <int BLOCK>
__device__ __forceinline__ void medium_sort(uint32_t *&k, uint32_t *&kt, uint32_t n,
                                            const SortPlan &sp, unsigned char *raw,
                                            MediumTail<BLOCK> &T) {
    using namespace tc_small;
    constexpr uint32_t ST = Medium<BLOCK>::ST;
    uint32_t *xchg = reinterpret_cast<uint32_t *>(raw);
    uint32_t(*wcnt)[RADIX] = reinterpret_cast<uint32_t(*)[RADIX]>(raw + 4 * (size_t)ST);
    const int tid = threadIdx.x, w = tid / TC_WAVE;
    for (int p = 0; p < sp.passes; ++p) {
        uint32_t *base = T.hist[p];
        uint32_t all;
        const uint32_t c0 = tid < RADIX ? base[tid] : 0u;
        const uint32_t b0 = wg_scan<BLOCK>(c0, &all, T.wsum);
        if (tid < RADIX) base[tid] = b0;
        const int sh = sp.at(p), wd = sp.bits_at(p);
        const uint32_t mask = (1u << wd) - 1u;
        for (uint32_t t0 = 0; t0 < n; t0 += ST) {
            const uint32_t tn = n - t0 < ST ? n - t0 : ST;
            const int itn = (int)((tn + BLOCK - 1) / BLOCK);
            uint32_t key[ITEMS], place[ITEMS];
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) {
                const uint32_t i = elem(it, itn);
                key[it] = it < itn && i < tn ? at(k, t0 + i) : NONE;
            }
            digit_ranks<BLOCK, ITEMS>(key, itn, sh, wd, place, wcnt);
            __syncthreads();
            const uint32_t cnt = digit_starts<BLOCK>(wcnt, T.wsum);
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
                if (it < itn) xchg[place[it] + wcnt[w][(key[it] >> sh) & mask]] = key[it];
            __syncthreads();
            // absent places (all ones) are last in the tile
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) {
                const uint32_t i = it * BLOCK + tid;
                if (i < tn) {
                    const uint32_t x = xchg[i], d = (x >> sh) & mask;
                    at(kt, base[d] + i - wcnt[0][d]) = x;
                }
            }
            __syncthreads();
            if (tid < RADIX) base[tid] += cnt;
        }
        __syncthreads();
        uint32_t *t = k;
        k = kt;
        kt = t;
    }
}

// An oriented edge on its way to its row.
struct alignas(4) Entry {
    uint32_t ends, edge;
};

template <int BLOCK>
__device__ __forceinline__ void fused_medium(const FusedArgs &a, const GraphRef q, unsigned char *raw,
                             MediumTail<BLOCK> &T) {
    using namespace tc_small;
    constexpr uint32_t NMAX = Medium<BLOCK>::NMAX, LT = Medium<BLOCK>::LT, CT = Medium<BLOCK>::CT, HALO = Medium<BLOCK>::HALO;
    constexpr int U = 8;  // elements per thread of a tile
    const uint32_t n = q.n, P = q.P;
    const int tid = threadIdx.x;
    // the graph's own slices
    const uint32_t *const src = reinterpret_cast<const uint32_t *>(a.src) + q.pa;
    const uint32_t *const dst = reinterpret_cast<const uint32_t *>(a.dst) + q.pa;
    const int b = bits_of(n > 1 ? n - 1 : 1);
    const uint32_t none = (uint32_t)((1ull << (2 * b)) - 1ull), vm = (1u << b) - 1u;
    uint32_t *const words = reinterpret_cast<uint32_t *>(raw);        // one per vertex
    uint32_t *const second = reinterpret_cast<uint32_t *>(raw) + NMAX;  // after them
    for (int i = tid; i < 4 * RADIX; i += BLOCK) (&T.hist[0][0])[i] = 0;
    __syncthreads();
    // keys lo << b | hi (self-loops all ones), with the id range check and the
    // digit counts of their sort
    const SortPlan kp(0, 2 * b);
    bool bad = false;
    for (uint32_t t0 = 0; t0 < P; t0 += LT) {
        uint32_t x[U], y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = t0 + u * BLOCK + tid;
            x[u] = i < P ? at(src, i) : 0u;
            y[u] = i < P ? at(dst, i) : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = t0 + u * BLOCK + tid;
            if (i < P) {
                uint32_t key = none;
                if (x[u] >= n || y[u] >= n) bad = true;
                else if (x[u] != y[u]) key = x[u] < y[u] ? x[u] << b | y[u] : y[u] << b | x[u];
                at(q.A, i) = key;
                medium_hist<BLOCK>(kp, key, T);
            }
        }
    }
    if (wg_any(bad)) {
        fused_fail<BLOCK>(a, q.g, q.va, n, TC_ERR_VERTEX_RANGE);
        return;
    }
    uint32_t *k = q.A, *kt = q.B;
    medium_sort<BLOCK>(k, kt, P, kp, raw, T);
    // canonical edges (to C, and eu / ev) with the degrees in LDS
    for (uint32_t v = tid; v < n; v += BLOCK) words[v] = 0;
    __syncthreads();
    uint32_t m = 0;
    for (uint32_t t0 = 0; t0 < P; t0 += LT) {
        uint32_t key[U], prev[U], pos[U];
        bool keep[U];
        uint32_t mine = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = t0 + elem(u, U);
            key[u] = i < P ? at(k, i) : none;
            prev[u] = i > 0 && i < P ? at(k, i - 1) : none;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            keep[u] = key[u] != none && prev[u] != key[u];
            const uint64_t bal = __ballot(keep[u]);
            pos[u] = mine + (uint32_t)__popcll(bal & tc_lanemask_lt());
            mine += (uint32_t)__popcll(bal);
        }
        uint32_t all;
        const uint32_t first = wg_scan<BLOCK>(__lane_id() == 0 ? mine : 0u, &all, T.wsum);
        const uint32_t base = m + __shfl(first, 0, TC_WAVE);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (keep[u]) {
                const uint32_t e = base + pos[u], lo = key[u] >> b, hi = key[u] & vm;
                at(q.C, e) = key[u];
                if (a.eu) at(a.eu + q.pa, e) = (int32_t)lo;
                if (a.ev) at(a.ev + q.pa, e) = (int32_t)hi;
                atomicAdd(&words[lo], 1u);
                atomicAdd(&words[hi], 1u);
            }
        m += all;
    }
    __syncthreads();
    // order (degree, id): degree << 16 | id, stable on the degree's bits
    uint32_t dmax = 0;
    for (uint32_t v = tid; v < n; v += BLOCK) dmax = words[v] > dmax ? words[v] : dmax;
    dmax = wg_max<BLOCK>(dmax, T.wsum);
    const SortPlan rp(16, bits_of(dmax));
    for (int i = tid; i < 4 * RADIX; i += BLOCK) (&T.hist[0][0])[i] = 0;
    __syncthreads();
    for (uint32_t v = tid; v < n; v += BLOCK) {
        const uint32_t key = words[v] << 16 | v;
        at(q.deg, v) = key;
        medium_hist<BLOCK>(rp, key, T);
    }
    __syncthreads();
    k = q.deg;
    kt = q.vtmp;
    medium_sort<BLOCK>(k, kt, n, rp, raw, T);
    uint16_t *const rank = reinterpret_cast<uint16_t *>(second);
    for (uint32_t v = tid; v < n; v += BLOCK) words[v] = 0;
    for (uint32_t r = tid; r < n; r += BLOCK) {
        const uint32_t v = at(k, r) & 0xFFFFu;
        rank[v] = (uint16_t)r;
        at(q.rank, v) = r;
    }
    __syncthreads();
    // orientation: row lengths, their offsets as cursors, then every edge into
    // its row as (lower rank << 16 | higher rank, edge), any order: one 8-byte
    // store per edge (A and B), since each store of the scatter is a sector
    Entry *const entry = reinterpret_cast<Entry *>(q.A);
    uint32_t longest = 0;  // row
    for (int pass = 0; pass < 2; ++pass) {
        for (uint32_t t0 = 0; t0 < m; t0 += LT) {
            uint32_t key[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t e = t0 + u * BLOCK + tid;
                key[u] = e < m ? at(q.C, e) : 0u;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t e = t0 + u * BLOCK + tid;
                if (e < m) {
                    const uint32_t x = rank[key[u] >> b], y = rank[key[u] & vm];
                    const uint32_t r = x < y ? x : y, h = x < y ? y : x;
                    const uint32_t s = atomicAdd(&words[r], 1u);
                    if (pass == 1) {
                        at(entry, s) = Entry{r << 16 | h, e};
                    }
                }
            }
        }
        __syncthreads();
        if (pass == 0) {
            constexpr int PER = (int)(NMAX / BLOCK);
            uint32_t sum = 0, all;
            const uint32_t r0 = tid * PER;
            for (int j = 0; j < PER; ++j) {
                const uint32_t d = r0 + j < n ? words[r0 + j] : 0u;
                sum += d;
                longest = d > longest ? d : longest;
            }
            longest = wg_max<BLOCK>(longest, T.wsum);
            uint32_t off = wg_scan<BLOCK>(sum, &all, T.wsum);
            for (int j = 0; j < PER; ++j)
                if (r0 + j < n) {
                    const uint32_t d = words[r0 + j];
                    words[r0 + j] = off;
                    off += d;
                }
            __syncthreads();
        }
    }
    // words[r] is now the end of row r.  Each row in order of the higher rank:
    // an entry's place is the number of smaller ones in its row, counted in an
    // LDS copy of the tile and the rows that reach into it
    const auto row_start = [&](uint32_t r) { return r > 0 ? words[r - 1] : 0u; };
    uint32_t *const tile = second, *const ocol = q.D, *const o2e = q.E;
    for (uint32_t t0 = 0; t0 < m; t0 += LT) {
        const uint32_t lo = t0 > HALO ? t0 - HALO : 0u;
        const uint32_t hi = m - t0 > LT + HALO ? t0 + LT + HALO : m;
        for (uint32_t i = lo + tid; i < hi; i += BLOCK) tile[i - lo] = at(entry, i).ends;
        uint32_t e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t s = t0 + u * BLOCK + tid;
            e[u] = s < m ? at(entry, s).edge : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t s = t0 + u * BLOCK + tid;
            if (s < m) {
                const uint32_t me = tile[s - lo], r = me >> 16;
                const uint32_t ra = row_start(r), re = words[r];
                uint32_t to = ra;
                for (uint32_t i = ra; i < re; ++i) to += tile[i - lo] < me ? 1u : 0u;
                at(ocol, to) = me;
                at(o2e, to) = e[u];
            }
        }
        __syncthreads();
    }
    // count: the tail of N_H(r) after c merged with N_H(c), supports added to
    // the slots.  Added to the canonical edges, every hit outside LDS waits for
    // its slot's edge first: 16 complete graphs of 1000 vertices took 480 / 574 /
    // 701 ms at 1024 / 512 / 256 threads so, 318 / 373 / 478 now; with no graph in
    // LDS (fused_large) 427 / 407 / 384.  A lane goes on to its next slot as soon as
    // its merge ends, without waiting for the longest merge of the wavefront.  The
    // last slots, whose rows are of the highest ranks and merged most, lie in LDS
    // with their counts (column | count << 16; a support is below n < 2^16), the
    // others are taken in tiles that do while they are a merge's own row: what is
    // left to device memory are the rows N_H(c) of lower ranks and their hits.  The
    // edges' supports are cleared in order first and only those above 0 scattered
    // afterwards (each such store is a sector: all of them scattered made the batch
    // of 4096 BA graphs 11.1 ms, 10.1 so, 10.6 with supports on the edges)
    uint32_t *const osup = q.A;  // the entries are no longer needed
    for (uint32_t s = tid; s < m; s += BLOCK) {
        at(osup, s) = 0;
        if (a.sup) at(a.sup + q.pa, s) = 0;
    }
    uint32_t *const top = words + n;
    const uint32_t room = (uint32_t)(Medium<BLOCK>::BYTES / 4) - n - Medium<BLOCK>::PAD;
    const uint32_t kept = m <= room ? m : room - (CT + longest), top0 = m - kept;
    uint32_t *const run = top + kept;
    for (uint32_t i = tid; i < kept; i += BLOCK) top[i] = at(ocol, top0 + i) & 0xFFFFu;
    __syncthreads();
    for (uint32_t t0 = 0; t0 < m; t0 = t0 < top0 ? (top0 - t0 > CT ? t0 + CT : top0) : m) {
        const bool tile = t0 < top0;
        const uint32_t end = tile ? (top0 - t0 > CT ? t0 + CT : top0) : m;
        uint32_t *const own = tile ? run : top;  // slot t0 on
        const uint32_t len = (m - end > longest && tile ? end + longest : m) - t0;
        if (tile) {
            for (uint32_t i = tid; i < len; i += BLOCK) own[i] = at(ocol, t0 + i) & 0xFFFFu;
            __syncthreads();
        }
        uint32_t s = t0 + tid, t = 0, i = 0, ie = 0, j = 0, je = 0;
        uint32_t w = s < end ? at(ocol, s) : 0u;
        bool open = false;  // slot s is being merged
        for (;;) {
            while (s < end && !(open && i < ie && j < je)) {
                if (open) {
                    if (t) atomicAdd(&own[s - t0], t << 16);
                    s += BLOCK;
                    if (s >= end) break;
                    w = at(ocol, s);
                }
                const uint32_t c = w & 0xFFFFu;
                i = s + 1;
                ie = words[w >> 16];
                j = row_start(c);
                je = words[c];
                t = 0;
                open = true;
            }
            if (s >= end) break;
            // windows may reach past their row, and past the last one into
            // what follows
            uint32_t x[8], y[8], na, nb, hits, where;
            const bool in_top = j >= top0;
            if (in_top) {
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = top[j - top0 + e];
            } else {
                load8(&at(ocol, j), y);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = own[i - t0 + e];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                x[e] &= 0xFFFFu;
                y[e] &= 0xFFFFu;
            }
            merge_round(x, y, ie - i, je - j, na, nb, hits, where);
            t += (uint32_t)__popc(hits);
            while (hits) {
                const uint32_t e = (uint32_t)__ffs((int)hits) - 1u;
                const uint32_t f = j + ((where >> (4 * e)) & 15u);
                hits &= hits - 1u;
                atomicAdd(&own[i - t0 + e], 1u << 16);
                if (in_top) atomicAdd(&top[f - top0], 1u << 16);
                else wg_add(&at(osup, f), 1u);
            }
            i += na;
            j += nb;
        }
        __syncthreads();
        for (uint32_t i = tid; i < len; i += BLOCK) {
            const uint32_t c = own[i] >> 16;
            if (c) wg_add(&at(osup, t0 + i), c);
        }
        __syncthreads();
    }
    // twice the triangles per rank, in LDS, with the supports out.  32 bits hold
    // every sum here: at most 2^20 edges make at most T = 5.1e8 triangles, and a
    // vertex's weighted sum is at most 3 T as well.  Its neighbours of weight 3 are
    // adjacent to none of its other neighbours (that would be a triangle), so a
    // triangle with one of them has no second neighbour among its vertices and
    // counts 3; the others have at most three neighbours of weight 1
    for (uint32_t r = tid; r < n; r += BLOCK) words[r] = 0;
    __syncthreads();
    uint32_t local = 0;
    for (uint32_t t0 = 0; t0 < m; t0 += LT) {
        uint32_t ends[U], x[U], e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t s = t0 + u * BLOCK + tid;
            ends[u] = s < m ? at(ocol, s) : 0u;
            x[u] = s < m ? at(osup, s) : 0u;
            e[u] = s < m && a.sup ? at(o2e, s) : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (x[u]) {
                if (a.sup) at(a.sup + q.pa, e[u]) = x[u];
                atomicAdd(&words[ends[u] >> 16], x[u]);
                atomicAdd(&words[ends[u] & 0xFFFFu], x[u]);
                local += x[u];
            }
        }
    }
    const uint32_t three_t = wg_sum<BLOCK>(local, T.wsum);  // has the barrier
    bool odd = three_t % 3 != 0;
    uint32_t *const tri = reinterpret_cast<uint32_t *>(q.triR);
    for (uint32_t r = tid; r < n; r += BLOCK) {
        const uint32_t t2 = words[r];
        odd |= (t2 & 1u) != 0;
        at(tri, r) = t2 >> 1;
        words[r] = 0;
    }
    __syncthreads();
    // numerator: weight 1 for triangle neighbours (support > 0), 3 for others
    for (uint32_t t0 = 0; t0 < m; t0 += LT) {
        uint32_t ends[U], x[U], tl[U], th[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t s = t0 + u * BLOCK + tid;
            ends[u] = s < m ? at(ocol, s) : 0u;
            x[u] = s < m ? at(osup, s) : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            tl[u] = at(tri, ends[u] >> 16);
            th[u] = at(tri, ends[u] & 0xFFFFu);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t s = t0 + u * BLOCK + tid;
            if (s < m) {
                const uint32_t f = x[u] ? 1u : 3u;
                if (th[u]) atomicAdd(&words[ends[u] >> 16], f * th[u]);
                if (tl[u]) atomicAdd(&words[ends[u] & 0xFFFFu], f * tl[u]);
            }
        }
    }
    __syncthreads();
    const uint64_t tg = three_t / 3;
    for (uint32_t v = tid; v < n; v += BLOCK) {
        const uint32_t r = at(q.rank, v);
        const uint64_t t = at(tri, r), x = words[r] + t;
        if (a.tri) a.tri[q.va + v] = t;
        if (a.num) a.num[q.va + v] = x;
        if (a.tc) a.tc[q.va + v] = tg == 0 ? 0.0 : __ddiv_rn((double)x, (double)(3 * tg));
    }
    odd = wg_any(odd);
    if (tid == 0) {
        a.num_edges[q.g] = m;
        if (a.triG) a.triG[q.g] = tg;
        a.status[q.g] = odd ? TC_ERR_DEVICE : (tg == 0 ? TC_TRIANGLE_FREE : TC_OK);
    }
}

// ---------------------------------------------------------------------------
// Every other graph (more vertices than LDS holds, or more pairs): all arrays
// in the workspace.
// ---------------------------------------------------------------------------
template <int BLOCK>
__device__ __forceinline__ void fused_large(const FusedArgs &a, const GraphRef q, FusedLds<BLOCK> &sh) {
    const int tid = threadIdx.x;
    const int32_t g = q.g;
    const int64_t pa = q.pa, va = q.va;
    const uint32_t n = q.n, P = q.P;
    const uint32_t sentinel = n * n;  // n <= 65535: below 2^32
    uint32_t *A = q.A, *B = q.B, *C = q.C, *D = q.D, *E = q.E;
    uint64_t *triR = q.triR, *numR = q.numR;
    uint32_t *deg = q.deg, *rank = q.rank, *perm = q.perm, *vtmp = q.vtmp, *orp = q.orp;

    // keys, with the id range check
    bool bad = false;
    for (uint32_t i = tid; i < P; i += BLOCK) {
        const int32_t x = a.src[pa + i], y = a.dst[pa + i];
        uint32_t key = sentinel;
        if ((uint32_t)x >= n || (uint32_t)y >= n) {
            bad = true;
        } else if (x != y) {
            const uint32_t lo = (uint32_t)(x < y ? x : y), hi = (uint32_t)(x < y ? y : x);
            key = lo * n + hi;
        }
        A[i] = key;
    }
    if (wg_any(bad)) {
        fused_fail<BLOCK>(a, g, va, n, TC_ERR_VERTEX_RANGE);
        return;
    }
    // canonical edges
    uint32_t *k = A, *kt = B, *nv = nullptr, *nvt = nullptr;
    block_sort<BLOCK, false>(k, kt, nv, nvt, P, fused_bits(sentinel), sh);
    const uint32_t m = block_unique<BLOCK>(k, P, sentinel, C, sh);
    if (a.eu || a.ev) {
        for (uint32_t e = tid; e < m; e += BLOCK) {
            const uint32_t key = C[e], lo = key / n, hi = key - lo * n;
            if (a.eu) a.eu[pa + e] = (int32_t)lo;
            if (a.ev) a.ev[pa + e] = (int32_t)hi;
        }
    }

    // degrees
    for (uint32_t v = tid; v < n; v += BLOCK) deg[v] = 0;
    __syncthreads();
    // canonical edges come sorted by their smaller end: a wavefront's lanes
    // with the same smaller end form a run, whose first lane adds its length
    for (uint32_t e0 = 0; e0 < m; e0 += BLOCK) {
        const uint32_t e = e0 + tid;
        const bool valid = e < m;
        uint32_t lo = 0, hi = 0;
        if (valid) {
            const uint32_t key = C[e];
            lo = key / n;
            hi = key - lo * n;
        }
        const int lane = __lane_id();
        const uint32_t prev = __shfl_up(lo, 1, TC_WAVE);
        const bool head = valid && (lane == 0 || prev != lo);
        const uint64_t heads = __ballot(head);
        const uint64_t live = __ballot(valid);
        if (head) {
            const uint64_t after = lane == TC_WAVE - 1 ? 0ull : (heads >> (lane + 1)) << (lane + 1);
            const uint32_t end = after ? (uint32_t)(__ffsll((unsigned long long)after) - 1)
                                       : (uint32_t)(64 - __clzll(live));
            wg_add(&deg[lo], end - (uint32_t)lane);
        }
        if (valid) wg_add(&deg[hi], 1u);
    }
    __syncthreads();
    // order (degree, id): keys d * n + v, sorted; the key gives v back
    uint32_t dmax = 0;
    for (uint32_t v = tid; v < n; v += BLOCK) {
        const uint32_t d = deg[v];
        dmax = d > dmax ? d : dmax;
        deg[v] = d * n + v;
    }
    dmax = block_max32<BLOCK>(dmax, sh);
    k = deg;
    kt = vtmp;
    block_sort<BLOCK, false>(k, kt, nv, nvt, n, n ? fused_bits(dmax * n + (n - 1)) : 0, sh);
    for (uint32_t r = tid; r < n; r += BLOCK) {
        const uint32_t key = k[r], v = key - (key / n) * n;
        perm[r] = v;
        rank[v] = r;
    }
    __syncthreads();

    // orientation: keys rank(low) * n + rank(high), values canonical edge
    for (uint32_t e = tid; e < m; e += BLOCK) {
        const uint32_t key = C[e], lo = key / n, hi = key - lo * n;
        const uint32_t ra = rank[lo], rb = rank[hi];
        A[e] = ra < rb ? ra * n + rb : rb * n + ra;
        D[e] = e;
    }
    for (uint32_t r = tid; r < n; r += BLOCK) {
        triR[r] = 0;
        numR[r] = 0;
    }
    __syncthreads();
    k = A;
    kt = B;
    uint32_t *o2e = D, *vt = E;
    block_sort<BLOCK, true>(k, kt, o2e, vt, m, n ? fused_bits(n * n - 1) : 0, sh);
    uint32_t *ocol = k, *orow = kt, *osup = vt;
    for (uint32_t s = tid; s < m; s += BLOCK) {
        const uint32_t key = ocol[s], r = key / n;
        orow[s] = r;
        ocol[s] = key - r * n;
        osup[s] = 0;
    }
    __syncthreads();
    // row offsets: every entry of orp[0..n] is written once.  A slot opens its row
    // and the empty ones before it; where these are many (the isolated vertices
    // come first) its wavefront writes them together.  256 graphs of 65000 vertices
    // and 1000 pairs: 2.7 to 3.4 ms with a thread for all of a slot's, by how that
    // loop came out of the compiler, 0.95 ms so
    for (uint32_t s0 = 0; s0 < m; s0 += BLOCK) {
        const uint32_t s = s0 + tid;
        uint32_t from = 0, end = 0;
        if (s < m) {
            from = s == 0 ? 0u : orow[s - 1] + 1u;
            end = orow[s] + 1u;
        }
        uint64_t wide = __ballot(end > from + TC_WAVE);
        if (end <= from + TC_WAVE)
            for (uint32_t q = from; q < end; ++q) orp[q] = s;
        while (wide) {
            const int l = __ffsll((unsigned long long)wide) - 1;
            wide &= wide - 1;
            const uint32_t e = __shfl(end, l, TC_WAVE), x = __shfl(s, l, TC_WAVE);
            for (uint32_t q = __shfl(from, l, TC_WAVE) + __lane_id(); q < e; q += TC_WAVE) orp[q] = x;
        }
    }
    for (uint32_t q = (m > 0 ? orow[m - 1] + 1u : 0u) + tid; q <= n; q += BLOCK) orp[q] = m;
    __syncthreads();

    // count: the tail of N_H(r) after c against N_H(c), merged eight entries of
    // each list at a time: the sixteen loads of a round are independent (one
    // memory latency per round instead of one per step), all 64 pairs are
    // compared, and every entry up to the smaller of the two windows' last
    // entries is then settled (an entry above it can equal nothing in the other
    // window)
    for (uint32_t s = tid; s < m; s += BLOCK) {
        const uint32_t r = orow[s], c = ocol[s];
        uint32_t i = s + 1, j = orp[c];
        const uint32_t ie = orp[r + 1], je = orp[c + 1];
        uint32_t t = 0;
        while (i < ie && j < je) {
            uint32_t x[FUSED_MW], y[FUSED_MW];
#pragma unroll
            for (int e = 0; e < FUSED_MW; ++e) x[e] = i + e < ie ? ocol[i + e] : 0xFFFFFFFFu;
#pragma unroll
            for (int e = 0; e < FUSED_MW; ++e) y[e] = j + e < je ? ocol[j + e] : 0xFFFFFFFEu;
            const uint32_t lim = x[FUSED_MW - 1] < y[FUSED_MW - 1] ? x[FUSED_MW - 1] : y[FUSED_MW - 1];
            uint32_t na = 0, nb = 0;
#pragma unroll
            for (int e = 0; e < FUSED_MW; ++e) {
                na += x[e] <= lim ? 1u : 0u;
                nb += y[e] <= lim ? 1u : 0u;
            }
#pragma unroll
            for (int e = 0; e < FUSED_MW; ++e) {
                int f = -1;  // the other window's entry equal to x[e], if any
#pragma unroll
                for (int q = 0; q < FUSED_MW; ++q) f = x[e] == y[q] ? q : f;
                if (f >= 0) {
                    wg_add(&osup[i + e], 1u);
                    wg_add(&osup[j + f], 1u);
                    ++t;
                }
            }
            i += na;
            j += nb;
        }
        if (t) wg_add(&osup[s], t);
    }
    __syncthreads();

    // tri(v) = 1/2 Σ sup over v's edges; 3 triG = Σ_e sup(e)
    // (slots are sorted by row: a wavefront's slots of one row form a run)
    uint64_t local = 0;
    for (uint32_t s0 = 0; s0 < m; s0 += BLOCK) {
        const uint32_t s = s0 + tid;
        const bool valid = s < m;
        const uint32_t x = valid ? osup[s] : 0u, r = valid ? orow[s] : 0u;
        bool tail;
        const uint64_t rs = run_sum(r, (uint64_t)x, valid, tail);
        if (tail && rs) wg_add(&triR[r], rs);
        if (x) wg_add(&triR[ocol[s]], (uint64_t)x);
        local += x;
    }
    const uint64_t three_t = block_sum64<BLOCK>(local, sh);
    bool odd = (three_t % 3) != 0;
    for (uint32_t r = tid; r < n; r += BLOCK) {
        const uint64_t t2 = triR[r];
        odd |= (t2 & 1) != 0;
        triR[r] = t2 >> 1;
    }
    odd = __syncthreads_or(odd);
    const uint64_t tg = three_t / 3;

    // numerator: weight 1 for triangle neighbours (sup > 0), 3 for the others
    for (uint32_t s0 = 0; s0 < m; s0 += BLOCK) {
        const uint32_t s = s0 + tid;
        const bool valid = s < m;
        uint32_t r = 0, c = 0;
        uint64_t f = 0;
        if (valid) {
            r = orow[s];
            c = ocol[s];
            f = osup[s] ? 1 : 3;
        }
        bool tail;
        const uint64_t rs = run_sum(r, valid ? f * triR[c] : 0ull, valid, tail);
        if (tail && rs) wg_add(&numR[r], rs);
        if (valid) {
            const uint64_t y = f * triR[r];
            if (y) wg_add(&numR[c], y);
        }
    }
    __syncthreads();

    // outputs in the graph's own vertex ids and canonical edge order
    for (uint32_t r = tid; r < n; r += BLOCK) {
        const uint32_t v = perm[r];
        const uint64_t t = triR[r], x = numR[r] + t;
        if (a.tri) a.tri[va + v] = t;
        if (a.num) a.num[va + v] = x;
        if (a.tc) a.tc[va + v] = tg == 0 ? 0.0 : __ddiv_rn((double)x, (double)(3 * tg));
    }
    if (a.sup)
        for (uint32_t s = tid; s < m; s += BLOCK) a.sup[pa + o2e[s]] = osup[s];
    if (tid == 0) {
        a.num_edges[g] = m;
        if (a.triG) a.triG[g] = tg;
        a.status[g] = odd ? TC_ERR_DEVICE : (tg == 0 ? TC_TRIANGLE_FREE : TC_OK);
    }
}

// The caller has the barrier before the next graph.
template <int BLOCK>
__device__ __forceinline__ void fused_one_graph(const FusedArgs &a, int32_t g, FusedArena<BLOCK> &sh) {
    const int tid = threadIdx.x;
    const int64_t pa = a.pair_off[g], pb = a.pair_off[g + 1];
    const int64_t va = a.vtx_off[g], vb = a.vtx_off[g + 1];
    // offsets outside the arrays, or decreasing: nothing of this graph is
    // touched but its status
    if (pa < 0 || pb < pa || pb > a.P || va < 0 || vb < va || vb > a.N) {
        if (tid == 0) {
            a.num_edges[g] = 0;
            a.status[g] = TC_ERR_INVALID_ARG;
        }
        return;
    }
    if (vb - va > FUSED_MAX_N || pb - pa > 0x7FFFFFFFll) {
        fused_fail<BLOCK>(a, g, va, vb - va, TC_ERR_UNSUPPORTED);
        return;
    }
    GraphRef q;
    q.g = g;
    q.pa = pa;
    q.va = va;
    q.n = (uint32_t)(vb - va);
    q.P = (uint32_t)(pb - pa);
    // workspace of this graph: 5 pair arrays, then the vertex arrays
    q.A = reinterpret_cast<uint32_t *>(a.ws + FUSED_HEADER) + 5 * pa;
    q.B = q.A + q.P;
    q.C = q.B + q.P;
    q.D = q.C + q.P;
    q.E = q.D + q.P;
    unsigned char *vbase = a.ws + FUSED_HEADER + pair_region(a.P) + FUSED_VTX_BYTES * va +
                           FUSED_GRAPH_BYTES * (int64_t)g;
    q.triR = reinterpret_cast<uint64_t *>(vbase);
    q.numR = q.triR + q.n;
    q.deg = reinterpret_cast<uint32_t *>(q.numR + q.n);
    q.rank = q.deg + q.n;
    q.perm = q.rank + q.n;
    q.vtmp = q.perm + q.n;
    q.orp = q.vtmp + q.n;
    if (q.P <= (uint32_t)tc_small::Lds<BLOCK>::CAP && q.n <= (uint32_t)tc_small::Lds<BLOCK>::NMAX)
        fused_small<BLOCK>(a, q, sh.small);
    else if (q.P <= Medium<BLOCK>::PMAX && q.n <= Medium<BLOCK>::NMAX)
        fused_medium<BLOCK>(a, q, sh.medium.raw, sh.medium.tail);
    else
        fused_large<BLOCK>(a, q, sh.large);
}

__global__ void k_fused_init(unsigned char *ws) {
    if (threadIdx.x == 0) reinterpret_cast<uint32_t *>(ws)[0] = 0;
}

// Wavefronts per SIMD that a workgroup size asks for.  512 threads: 4 (at most
// 128 VGPRs), so that two workgroups fit on a compute unit.  256: 3 (168), for the
// three that LDS holds; with the 212 that the tiers take if left alone it is two,
// and 600 graphs of 30000 vertices and 120000 pairs take 18.9 ms (16.3 so), 3000
// BA graphs of 60 to 260 vertices 0.19 (0.15), but 4096 BA graphs of up to 20000
// vertices 32.6 (35.3); before the tiers, with 4 per SIMD, the three took 16.2,
// 0.43 and 38.3 ms.
constexpr int fused_waves(int block) { return block == 512 ? 4 : block == 256 ? 3 : 1; }

template <int BLOCK>
__global__ __launch_bounds__(BLOCK, fused_waves(BLOCK)) void k_fused_graphs(FusedArgs a) {
    __shared__ FusedArena<BLOCK> sh;
    __shared__ uint32_t next;
    uint32_t *head = reinterpret_cast<uint32_t *>(a.ws);
    for (;;) {
        if (threadIdx.x == 0) next = atomicAdd(head, 1u);
        __syncthreads();
        // the same value in every lane: keep it (and what derives from it) in
        // scalar registers
        const uint32_t slot = __builtin_amdgcn_readfirstlane(next);
        if (slot >= (uint32_t)a.G) break;
        const int32_t g = a.order ? __builtin_amdgcn_readfirstlane(a.order[slot]) : (int32_t)slot;
        // not a permutation: skip the entry
        if (g >= 0 && g < a.G) fused_one_graph<BLOCK>(a, g, sh);
        // Every way through the loop ends at this barrier.  A refused graph ends
        // with thread 0's stores, and with nothing between them and the fetch
        // above the compiler joins the two tests of threadIdx.x == 0: the other
        // lanes then go round a loop of their own, in which thread 0 never
        // fetches again, and the launch does not end.
        __syncthreads();
    }
}

int cu_count() {
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cus[dev] == 0) {
        int c = 0;
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0)
            c = 256;
        cus[dev] = c;
    }
    return cus[dev];
}

template <int BLOCK>
tc_status launch(const FusedArgs &a, int wg_per_cu, hipStream_t s) {
    int64_t grid = (int64_t)cu_count() * wg_per_cu;
    if (grid > a.G) grid = a.G;
    if (grid < 1) grid = 1;
    k_fused_graphs<BLOCK><<<(unsigned)grid, BLOCK, 0, s>>>(a);
    TC_LAUNCHED();
    return TC_OK;
}

// Workspace of the allocation-free entry point: one array per GPU, held from
// the library's load to the end of the process and shared by every call on
// that GPU.  Host code never uses the array's name as an address (it is a
// host-side stand-in): the device address comes from hipGetSymbolAddress,
// taken once per device on the first call there, with that device current.
constexpr int64_t FUSED_SCRATCH_BYTES = (int64_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[FUSED_SCRATCH_BYTES];

std::mutex g_scratch_mu;
void *g_scratch_ptr[64] = {nullptr};

tc_status scratch_address(void **out) {
    int dev = 0;
    TC_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return TC_ERR_DEVICE;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        TC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return TC_ERR_DEVICE;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return TC_OK;
}

tc_status check_args(const int32_t *src, const int32_t *dst, const int64_t *pair_off,
                     const int64_t *vtx_off, int32_t G, int64_t P, int64_t N, const int64_t *num_edges,
                     const int32_t *status, const tc_fused_tuning *t) {
    if (G < 0 || P < 0 || N < 0) return TC_ERR_INVALID_ARG;
    if (G > 0 && (!pair_off || !vtx_off || !num_edges || !status)) return TC_ERR_INVALID_ARG;
    if (P > 0 && (!src || !dst)) return TC_ERR_INVALID_ARG;
    if (P >= (int64_t)1 << 40 || N >= (int64_t)1 << 40) return TC_ERR_UNSUPPORTED;
    if (t) {
        if (t->block != 256 && t->block != 512 && t->block != 1024) return TC_ERR_INVALID_ARG;
        if (t->wg_per_cu < 1 || t->wg_per_cu > 16) return TC_ERR_INVALID_ARG;
    }
    return TC_OK;
}

tc_status run(const int32_t *src, const int32_t *dst, const int64_t *pair_off,
              const int64_t *vtx_off, const int32_t *order, int32_t G, int64_t P, int64_t N,
              int32_t *eu, int32_t *ev, uint64_t *support, int64_t *num_edges, uint64_t *tri,
              uint64_t *triG, uint64_t *num, double *tc, int32_t *status, void *ws,
              const tc_fused_tuning *t, hipStream_t s) {
    if (G == 0) return TC_OK;
    FusedArgs a;
    a.src = src;
    a.dst = dst;
    a.pair_off = pair_off;
    a.vtx_off = vtx_off;
    a.order = order;
    a.G = G;
    a.P = P;
    a.N = N;
    a.eu = eu;
    a.ev = ev;
    a.sup = support;
    a.num_edges = num_edges;
    a.tri = tri;
    a.num = num;
    a.tc = tc;
    a.triG = triG;
    a.status = status;
    a.ws = static_cast<unsigned char *>(ws);
    tc_fused_tuning d;
    tc_fused_tuning_default(&d);
    const tc_fused_tuning &u = t ? *t : d;
    k_fused_init<<<1, 64, 0, s>>>(a.ws);
    TC_LAUNCHED();
    switch (u.block) {
        case 256: return launch<256>(a, u.wg_per_cu, s);
        case 512: return launch<512>(a, u.wg_per_cu, s);
        default: return launch<1024>(a, u.wg_per_cu, s);
    }
}

}  // namespace

extern "C" {

tc_status tc_fused_tuning_default(tc_fused_tuning *t) {
    if (!t) return TC_ERR_INVALID_ARG;
    // measured on MI355X, the 4096-graph BA batch (ms) and five ER graphs of 10 k
    // pairs (us): 1024 threads x 1 per compute unit 10.1, 103; 512 x 1 20.4, 186;
    // 512 x 2 22.4, 188; 256 x 4 35.3, 307.  Thousands of graphs of a few hundred
    // vertices go faster with more workgroups: 3000 of 60 to 260 vertices 343 us at
    // 1024 x 1, 195 at 512 x 2, 152 at 256 x 4.
    t->block = 1024;
    t->wg_per_cu = 1;
    return TC_OK;
}

int64_t tc_batch_fused_workspace_bytes(int64_t num_pairs, int64_t num_vertices, int32_t num_graphs) {
    if (num_pairs < 0 || num_vertices < 0 || num_graphs < 0) return -1;
    return FUSED_HEADER + pair_region(num_pairs) + FUSED_VTX_BYTES * num_vertices +
           FUSED_GRAPH_BYTES * (int64_t)num_graphs;
}

tc_status tc_batch_fused(const int32_t *src, const int32_t *dst, const int64_t *graph_pair_off,
                         const int64_t *graph_vtx_off, const int32_t *order, int32_t num_graphs,
                         int64_t num_pairs, int64_t num_vertices, int32_t *eu, int32_t *ev,
                         uint64_t *support, int64_t *num_edges, uint64_t *tri, uint64_t *triG,
                         uint64_t *num, double *tc, int32_t *status, void *workspace,
                         int64_t workspace_bytes, const tc_fused_tuning *tuning, void *stream) {
    TC_TRY(check_args(src, dst, graph_pair_off, graph_vtx_off, num_graphs, num_pairs, num_vertices,
                      num_edges, status, tuning));
    if (num_graphs == 0) return TC_OK;
    const int64_t need = tc_batch_fused_workspace_bytes(num_pairs, num_vertices, num_graphs);
    if (!workspace || workspace_bytes < need) return TC_ERR_INVALID_ARG;
    if (((uintptr_t)workspace & 255) != 0) return TC_ERR_INVALID_ARG;
    return run(src, dst, graph_pair_off, graph_vtx_off, order, num_graphs, num_pairs, num_vertices,
               eu, ev, support, num_edges, tri, triG, num, tc, status, workspace, tuning,
               (hipStream_t)stream);
}

int64_t tc_batch_fused_noalloc_max_bytes(void) { return FUSED_SCRATCH_BYTES; }

tc_status tc_batch_fused_noalloc(const int32_t *src, const int32_t *dst,
                                 const int64_t *graph_pair_off, const int64_t *graph_vtx_off,
                                 const int32_t *order, int32_t num_graphs, int64_t num_pairs,
                                 int64_t num_vertices, int32_t *eu, int32_t *ev, uint64_t *support,
                                 int64_t *num_edges, uint64_t *tri, uint64_t *triG, uint64_t *num,
                                 double *tc, int32_t *status, const tc_fused_tuning *tuning,
                                 void *stream) {
    TC_TRY(check_args(src, dst, graph_pair_off, graph_vtx_off, num_graphs, num_pairs, num_vertices,
                      num_edges, status, tuning));
    if (num_graphs == 0) return TC_OK;
    const int64_t need = tc_batch_fused_workspace_bytes(num_pairs, num_vertices, num_graphs);
    if (need > FUSED_SCRATCH_BYTES) return TC_ERR_BUDGET;
    void *ws = nullptr;
    TC_TRY(scratch_address(&ws));
    return run(src, dst, graph_pair_off, graph_vtx_off, order, num_graphs, num_pairs, num_vertices,
               eu, ev, support, num_edges, tri, triG, num, tc, status, ws, tuning,
               (hipStream_t)stream);
}

}  // extern "C"
