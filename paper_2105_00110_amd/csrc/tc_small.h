// One workgroup, one small graph: the steps from pairs to oriented rows with
// everything in LDS and registers.  Shared by the fused batch launch and by the
// build of small single graphs.
//
// A graph of at most CAP = 16 BLOCK pairs over at most CAP / 4 vertices: every
// thread keeps up to 16 elements in registers (first pairs, then edges), LDS
// holds what the threads exchange (152 KB for 1024 threads).  A graph's arrays in device memory would
// cost a memory round trip per step, and one workgroup has too few wavefronts
// to cover it.
#pragma once

#include "tc_internal.h"

namespace tc_small {

constexpr int ITEMS = 16;  // elements per thread
constexpr int RADIX = 256;

template <int BLOCK>
struct Lds {
    static constexpr int CAP = ITEMS * BLOCK;  // pairs
    static constexpr int NMAX = CAP / 4;       // vertices
    static constexpr int WAVES = BLOCK / TC_WAVE;
    uint32_t xchg[CAP];      // sort exchange; then the slots, row << 16 | higher rank
    uint32_t cnt[CAP / 2];   // degrees; row cursors; packed 16-bit supports of the slots
    uint32_t tri[NMAX], num[NMAX];  // per-vertex sums
    union {
        uint32_t wcnt[WAVES][RADIX];   // digit counts per wavefront
        uint16_t orp[NMAX + 2];        // row offsets
    };
    uint16_t rank[NMAX];
    uint32_t wsum[WAVES + 1];
};

// Orders a wavefront's own LDS accesses across its lanes for the compiler (no
// instruction).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int bits_of(uint32_t max_value) {
    return max_value == 0 ? 1 : 32 - __clz(max_value);
}

// Exclusive prefix of x over the workgroup; *total = the sum.
template <int BLOCK>
__device__ __forceinline__ uint32_t wg_scan(uint32_t x, uint32_t *total, uint32_t *wsum) {
    constexpr int W = BLOCK / TC_WAVE;
    const int w = threadIdx.x / TC_WAVE;
    const uint32_t incl = tc_wave_incl_scan(x);
    if (__lane_id() == TC_WAVE - 1) wsum[w] = incl;
    __syncthreads();
    uint32_t before = incl - x, all = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const uint32_t y = wsum[q];
        before += q < w ? y : 0u;
        all += y;
    }
    __syncthreads();
    *total = all;
    return before;
}

// Sum of x over the workgroup.
template <int BLOCK>
__device__ __forceinline__ uint32_t wg_sum(uint32_t x, uint32_t *wsum) {
    x = tc_wave_sum(x);
    if (__lane_id() == 0) wsum[threadIdx.x / TC_WAVE] = x;
    __syncthreads();
    uint32_t all = 0;
#pragma unroll
    for (int q = 0; q < BLOCK / TC_WAVE; ++q) all += wsum[q];
    __syncthreads();
    return all;
}

template <int BLOCK>
__device__ __forceinline__ uint32_t wg_max(uint32_t x, uint32_t *wsum) {
    x = tc_wave_max(x);
    if (__lane_id() == 0) wsum[threadIdx.x / TC_WAVE] = x;
    __syncthreads();
    uint32_t m = 0;
#pragma unroll
    for (int q = 0; q < BLOCK / TC_WAVE; ++q) m = wsum[q] > m ? wsum[q] : m;
    __syncthreads();
    return m;
}

// Position of a thread's it-th element when a wavefront holds 64 per lane
// element, itn elements a lane.
__device__ __forceinline__ uint32_t elem(int it, int itn) {
    return ((uint32_t)(threadIdx.x / TC_WAVE) * (uint32_t)itn + (uint32_t)it) * TC_WAVE +
           (uint32_t)__lane_id();
}

// Ranks of a stable pass over the width-bit digit at shift: place[it] is the number
// of elements with the same digit that come before in the wavefront's own, and
// wcnt[w][d] the wavefront's count of digit d.  The caller has a barrier before
// and after.
//
// Ranks come from ballots: the lanes with the same digit form a mask, the rank
// is the count of lower lanes in it plus the wavefront's count so far.
template <int BLOCK, int IT>
__device__ __forceinline__ void digit_ranks(const uint32_t (&key)[IT], int itn, int shift, int width,
                                            uint32_t (&place)[IT], uint32_t (*wcnt)[RADIX]) {
    const int w = threadIdx.x / TC_WAVE, lane = __lane_id();
    const uint64_t lt = tc_lanemask_lt();
    const uint32_t mask = (1u << width) - 1u;
#pragma unroll
    for (int q = 0; q < RADIX / TC_WAVE; ++q) wcnt[w][q * TC_WAVE + lane] = 0;
    wave_sync();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        if (it < itn) {
            const uint32_t d = (key[it] >> shift) & mask;
            uint64_t peers = ~0ull;
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                if (b < width) {
                    const bool bit = (d >> b) & 1u;
                    const uint64_t bal = __ballot(bit);
                    peers &= bit ? bal : ~bal;
                }
            }
            const uint32_t prior = wcnt[w][d];
            place[it] = prior + (uint32_t)__popcll(peers & lt);
            wave_sync();
            if ((peers >> lane) == 1ull) wcnt[w][d] = prior + (uint32_t)__popcll(peers);
            wave_sync();
        }
    }
}

// Turns the wavefronts' digit counts into starts: wcnt[w][d] = base(d) + the
// counts of the wavefronts before w, base(d) the exclusive prefix of the digit
// totals.  Returns this thread's digit total (threads below RADIX).
template <int BLOCK>
__device__ __forceinline__ uint32_t digit_starts(uint32_t (*wcnt)[RADIX], uint32_t *wsum) {
    constexpr int W = BLOCK / TC_WAVE;
    static_assert(BLOCK >= RADIX, "one digit per thread");
    const int tid = threadIdx.x;
    uint32_t run = 0;
    if (tid < RADIX) {
#pragma unroll
        for (int q = 0; q < W; ++q) run += wcnt[q][tid];
    }
    uint32_t all;
    uint32_t at = wg_scan<BLOCK>(tid < RADIX ? run : 0u, &all, wsum);
    if (tid < RADIX) {
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const uint32_t c = wcnt[q][tid];
            wcnt[q][tid] = at;
            at += c;
        }
    }
    __syncthreads();
    return run;
}

// Stable sort of the BLOCK * itn keys in registers by the bits [shift, shift +
// bits), bits >= 1; xchg ends holding them in order.
template <int BLOCK, int IT>
__device__ __forceinline__ void sort_regs(uint32_t (&key)[IT], int itn, int shift, int bits,
                                          Lds<BLOCK> &L) {
    const int passes = (bits + 7) / 8;
    const int width = (bits + passes - 1) / passes;
    for (int p = 0; p < passes; ++p) {
        uint32_t place[IT];
        const int sh = shift + p * width;
        const int wd = width < shift + bits - sh ? width : shift + bits - sh;
        digit_ranks<BLOCK, IT>(key, itn, sh, wd, place, L.wcnt);
        __syncthreads();
        (void)digit_starts<BLOCK>(L.wcnt, L.wsum);
        const int w = threadIdx.x / TC_WAVE;
        const uint32_t mask = (1u << wd) - 1u;
#pragma unroll
        for (int it = 0; it < IT; ++it)
            if (it < itn) L.xchg[place[it] + L.wcnt[w][(key[it] >> sh) & mask]] = key[it];
        __syncthreads();
#pragma unroll
        for (int it = 0; it < IT; ++it)
            if (it < itn) key[it] = L.xchg[elem(it, itn)];
    }
    __syncthreads();
}

// Eight consecutive 32-bit words from a 4-byte aligned address, in two loads.
struct alignas(4) Words4 {
    uint32_t w[4];
};
__device__ __forceinline__ void load8(const uint32_t *p, uint32_t (&x)[8]) {
    const Words4 a = *reinterpret_cast<const Words4 *>(p);
    const Words4 b = *reinterpret_cast<const Words4 *>(p + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[e] = a.w[e];
        x[e + 4] = b.w[e];
    }
}

// One round of merging two ascending lists through windows of 8 entries, nx
// and ny of them inside their lists (the others are ignored).  Every entry up
// to the smaller of the windows' last ones is settled: na and nb entries (past
// a list's end: all 8).  hits: bit e set if x[e] is in the other window, at
// place (where >> 4e) & 15.
__device__ __forceinline__ void merge_round(uint32_t (&x)[8], uint32_t (&y)[8], uint32_t nx,
                                            uint32_t ny, uint32_t &na, uint32_t &nb, uint32_t &hits,
                                            uint32_t &where) {
#pragma unroll
    for (uint32_t e = 0; e < 8; ++e) {
        x[e] = e < nx ? x[e] : 0xFFFFFFFFu;
        y[e] = e < ny ? y[e] : 0xFFFFFFFEu;
    }
    const uint32_t lim = x[7] < y[7] ? x[7] : y[7];
    na = nb = hits = where = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        na += x[e] <= lim ? 1u : 0u;
        nb += y[e] <= lim ? 1u : 0u;
        uint32_t f = 8;
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) f = x[e] == y[q] ? q : f;
        hits |= f < 8 ? 1u << e : 0u;
        where |= f << (4 * e);
    }
}

constexpr uint32_t NONE = 0xFFFFFFFFu;

// The edges of a graph in registers: ends[it] = lower end << 16 | higher end
// (NONE: no edge at this place), tag[it] = the canonical edge's number, with its
// slot << 16 once the edges are oriented.
struct Edges {
    uint32_t ends[ITEMS];
    uint32_t tag[ITEMS];
};

// Pairs to canonical edges: sorted, self-loops and repeats dropped.  key[it] is
// lo << b | hi (b bits a vertex, lo < hi) or all ones in 2b bits (self-loop, or
// no pair at this place).  Returns the number of edges.
template <int BLOCK>
__device__ __forceinline__ uint32_t canonical(uint32_t (&key)[ITEMS], int itn, int b, Edges &E,
                                              Lds<BLOCK> &L) {
    const uint32_t none = (uint32_t)((1ull << (2 * b)) - 1ull);
    sort_regs<BLOCK, ITEMS>(key, itn, 0, 2 * b, L);
    const uint64_t lt = tc_lanemask_lt();
    uint32_t mine = 0;  // edges of this wavefront before the current element row
    uint32_t at[ITEMS];
    bool keep[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        keep[it] = false;
        at[it] = 0;
        if (it < itn) {
            const uint32_t i = elem(it, itn);
            keep[it] = key[it] != none && (i == 0 || L.xchg[i - 1] != key[it]);
            const uint64_t bal = __ballot(keep[it]);
            at[it] = mine + (uint32_t)__popcll(bal & lt);
            mine += (uint32_t)__popcll(bal);
        }
    }
    uint32_t m;
    // every lane of the wavefront holds the same count: lane 0 stands for it
    const uint32_t first = wg_scan<BLOCK>(__lane_id() == 0 ? mine : 0u, &m, L.wsum);
    const uint32_t base = __shfl(first, 0, TC_WAVE);
    const uint32_t vm = (1u << b) - 1u;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        E.ends[it] = keep[it] ? (key[it] >> b) << 16 | (key[it] & vm) : NONE;
        E.tag[it] = base + at[it];
    }
    return m;
}

// Degrees into L.cnt[0..n), then the order (degree, id): L.rank[v], and each
// thread's share of the permutation, perm(r, v).  Returns the largest degree.
template <int BLOCK, typename Perm>
__device__ __forceinline__ uint32_t degree_rank(const Edges &E, uint32_t n, Lds<BLOCK> &L, Perm perm) {
    constexpr int IT = Lds<BLOCK>::NMAX / BLOCK;
    for (uint32_t v = threadIdx.x; v < n; v += BLOCK) L.cnt[v] = 0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        if (E.ends[it] != NONE) {
            atomicAdd(&L.cnt[E.ends[it] >> 16], 1u);
            atomicAdd(&L.cnt[E.ends[it] & 0xFFFFu], 1u);
        }
    __syncthreads();
    // (degree << 16 | v) in the order of v: a stable sort on the degree's bits
    const int itn = (int)((n + BLOCK - 1) / BLOCK);
    uint32_t key[IT], dmax = 0;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        key[it] = NONE;
        if (it < itn) {
            const uint32_t v = elem(it, itn);
            if (v < n) {
                const uint32_t d = L.cnt[v];
                dmax = d > dmax ? d : dmax;
                key[it] = d << 16 | v;
            }
        }
    }
    dmax = wg_max<BLOCK>(dmax, L.wsum);
    sort_regs<BLOCK, IT>(key, itn, 16, bits_of(dmax), L);
#pragma unroll
    for (int it = 0; it < IT; ++it)
        if (it < itn) {
            const uint32_t r = elem(it, itn);
            if (r < n) {
                L.rank[key[it] & 0xFFFFu] = (uint16_t)r;
                perm(r, key[it] & 0xFFFFu);
            }
        }
    __syncthreads();
    return dmax;
}

// Orientation: E.ends becomes lower rank << 16 | higher rank, the high half of
// E.tag the edge's slot in the rows of higher-ordered neighbours (by row, then
// by higher rank), L.orp the row offsets (orp[n] = m), L.xchg[slot] = E.ends.
// Returns the longest row.
template <int BLOCK>
__device__ __forceinline__ uint32_t orient(Edges &E, uint32_t n, uint32_t m, Lds<BLOCK> &L) {
    constexpr int IT = Lds<BLOCK>::NMAX / BLOCK;
    for (uint32_t v = threadIdx.x; v < n; v += BLOCK) L.cnt[v] = 0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if (E.ends[it] != NONE) {
            const uint32_t a = L.rank[E.ends[it] >> 16], c = L.rank[E.ends[it] & 0xFFFFu];
            const uint32_t r = a < c ? a : c, h = a < c ? c : a;
            E.ends[it] = r << 16 | h;
            E.tag[it] |= atomicAdd(&L.cnt[r], 1u) << 16;  // place in the row, any order
        }
    }
    __syncthreads();
    // offsets: every thread scans its consecutive rows
    uint32_t d[IT], sum = 0, dmax = 0, total;
    const uint32_t r0 = threadIdx.x * IT;
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        d[k] = r0 + k < n ? L.cnt[r0 + k] : 0u;
        dmax = d[k] > dmax ? d[k] : dmax;
        sum += d[k];
    }
    uint32_t at = wg_scan<BLOCK>(sum, &total, L.wsum);
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        if (r0 + k < n) L.orp[r0 + k] = (uint16_t)at;
        at += d[k];
    }
    if (threadIdx.x == 0) L.orp[n] = (uint16_t)m;
    dmax = wg_max<BLOCK>(dmax, L.wsum);
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        if (E.ends[it] != NONE) L.xchg[L.orp[E.ends[it] >> 16] + (E.tag[it] >> 16)] = E.ends[it];
    __syncthreads();
    // each entry's place in its row: the number of smaller ones
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        if (E.ends[it] != NONE) {
            const uint32_t r = E.ends[it] >> 16, a = L.orp[r], e = L.orp[r + 1];
            uint32_t s = a;
            for (uint32_t t = a; t < e; ++t) s += L.xchg[t] < E.ends[it] ? 1u : 0u;
            E.tag[it] = (E.tag[it] & 0xFFFFu) | s << 16;
        }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        if (E.ends[it] != NONE) L.xchg[E.tag[it] >> 16] = E.ends[it];
    __syncthreads();
    return dmax;
}

// Support of slot s, a 16-bit half (a support is below the number of vertices).
template <int BLOCK>
__device__ __forceinline__ uint32_t support(uint32_t s, const Lds<BLOCK> &L) {
    return (L.cnt[s >> 1] >> (16 * (s & 1u))) & 0xFFFFu;
}

// Count on the m slots in L.xchg (rows at L.orp): the tail of N_H(r) after c
// merged with N_H(c) for every slot r -> c; supports in L.cnt.  Clears L.tri and
// L.num.  Ends with a barrier.
template <int BLOCK>
__device__ __forceinline__ void count_slots(uint32_t m, uint32_t n, Lds<BLOCK> &L) {
    constexpr int MW = 4;
    for (uint32_t i = threadIdx.x; i < (m + 1) / 2; i += BLOCK) L.cnt[i] = 0;
    for (uint32_t v = threadIdx.x; v < n; v += BLOCK) L.tri[v] = L.num[v] = 0;
    __syncthreads();
    const auto add = [&](uint32_t s, uint32_t x) {
        atomicAdd(&L.cnt[s >> 1], x << (16 * (s & 1u)));
    };
#pragma unroll 1
    for (uint32_t s = threadIdx.x; s < m; s += BLOCK) {
        const uint32_t r = L.xchg[s] >> 16, c = L.xchg[s] & 0xFFFFu;
        uint32_t i = s + 1, j = L.orp[c], t = 0;
        const uint32_t ie = L.orp[r + 1], je = L.orp[c + 1];
        while (i < ie && j < je) {
            uint32_t x[MW], y[MW];
#pragma unroll
            for (int e = 0; e < MW; ++e) {
                x[e] = L.xchg[i + e < ie ? i + e : i] & 0xFFFFu;
                y[e] = L.xchg[j + e < je ? j + e : j] & 0xFFFFu;
            }
#pragma unroll
            for (int e = 0; e < MW; ++e) {
                x[e] = i + e < ie ? x[e] : 0xFFFFFFFFu;
                y[e] = j + e < je ? y[e] : 0xFFFFFFFEu;
            }
            const uint32_t lim = x[MW - 1] < y[MW - 1] ? x[MW - 1] : y[MW - 1];
            uint32_t na = 0, nb = 0;
#pragma unroll
            for (int e = 0; e < MW; ++e) {
                na += x[e] <= lim ? 1u : 0u;
                nb += y[e] <= lim ? 1u : 0u;
                int f = -1;
#pragma unroll
                for (int p = 0; p < MW; ++p) f = x[e] == y[p] ? p : f;
                if (f >= 0) {
                    add(i + e, 1u);
                    add(j + (uint32_t)f, 1u);
                    ++t;
                }
            }
            i += na;
            j += nb;
        }
        if (t) add(s, t);
    }
    __syncthreads();
}

// Sums over every vertex's edges: L.tri = twice the triangles of each rank,
// L.num = Σ weight * triangles of the other end (1 on edges with support, 3 on
// the others).  All below 2^32: at most 16384 edges make at most 988000
// triangles.  Returns Σ supports, three times the graph's triangles.
template <int BLOCK>
__device__ __forceinline__ uint32_t slot_sums(uint32_t m, Lds<BLOCK> &L) {
    uint32_t local = 0;
    for (uint32_t s = threadIdx.x; s < m; s += BLOCK) {
        const uint32_t x = support(s, L);
        if (x) {
            atomicAdd(&L.tri[L.xchg[s] >> 16], x);
            atomicAdd(&L.tri[L.xchg[s] & 0xFFFFu], x);
            local += x;
        }
    }
    const uint32_t all = wg_sum<BLOCK>(local, L.wsum);  // has the barrier
    for (uint32_t s = threadIdx.x; s < m; s += BLOCK) {
        const uint32_t r = L.xchg[s] >> 16, c = L.xchg[s] & 0xFFFFu;
        const uint32_t f = support(s, L) ? 1u : 3u, tr = L.tri[r] >> 1, tc = L.tri[c] >> 1;
        if (tc) atomicAdd(&L.num[r], f * tc);
        if (tr) atomicAdd(&L.num[c], f * tr);
    }
    __syncthreads();
    return all;
}

}  // namespace tc_small
