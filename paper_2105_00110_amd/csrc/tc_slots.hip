// Count and aggregation for flat graphs: every oriented row is short, so no
// lookup table, transposition or bit matrix pays.
//
// One thread per oriented slot (r -> c) merges the tail of N_H(r) after c with
// N_H(c), both sorted: the appendix's Procedure 2 (low and middle vertices'
// higher-ordered sets intersected) with counts in place of marks.  Every
// common w is the triangle (r, c, w), found once from its lowest vertex; it
// adds 1 to the support of (r, w) and (c, w), and the slot's own support gains
// the number found.  The sums over a vertex's edges that Algorithm 2 needs run
// over the same slots: a slot contributes to its row, summed over the row's run
// of lanes, and by an atomic to its higher end.
//
// What bounds it: the merge is bound by the random rows N_H(c) (two lines a
// slot), the sums by the atomics on the higher ends.  The ends with many slots
// are the top ranks (ranks follow degrees), so each workgroup keeps the
// SLOT_TOP highest ranks in LDS and adds them once at its end; a hub then
// costs one atomic per workgroup and not one per edge (11 ns each on one word).
//
// Whole calls, from the middle pivot with its transposition sort, bit matrices
// and rank-space sums to this: 5 M uniform pairs over 1.25 M vertices 2593 to
// 1316 us, 512 BA graphs with 17.8 M edges 8774 to 4601 us (count 890 us, sums
// 500 and 580 us).
#include "tc_internal.h"

namespace {

constexpr int BK = 256;
constexpr int MW = 8;  // entries of each list per round of the merge
constexpr int SLOT_TOP = 2048;
constexpr unsigned SUM_BLOCKS = 1024;
using ull = unsigned long long;

static inline unsigned grid_for(int64_t n, unsigned most) {
    const int64_t g = tc_div_up(n, BK);
    return (unsigned)(g < 1 ? 1 : (g < most ? g : most));
}

__device__ __forceinline__ int32_t graph_of(const int64_t *__restrict__ vtx_off, int32_t G,
                                            int64_t v) {
    int32_t lo = 0, hi = G - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (vtx_off[mid] <= v) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Sum of x over each run of equal keys among the wavefront's lanes (keys
// non-decreasing, key < 0: not taking part); the run's last lane gets the sum
// and tail = true.
__device__ __forceinline__ uint64_t run_sum(int32_t key, uint64_t x, bool &tail) {
    const int lane = __lane_id();
#pragma unroll
    for (int off = 1; off < TC_WAVE; off <<= 1) {
        const uint64_t y = __shfl_up(x, off, TC_WAVE);
        const int32_t k = __shfl_up(key, off, TC_WAVE);
        if (lane >= off && k == key) x += y;
    }
    const int32_t next = __shfl_down(key, 1, TC_WAVE);
    tail = key >= 0 && (lane == TC_WAVE - 1 || next != key);
    return x;
}

// ocol is padded by TC_OCOL_PAD entries past the last row, so a window may be
// loaded whole; entries past a list's end are replaced by values that equal
// nothing.
__global__ __launch_bounds__(BK) void k_slot_count(int64_t m, const int64_t *__restrict__ orp,
                                                   const int32_t *__restrict__ ocol,
                                                   const int32_t *__restrict__ orow,
                                                   uint32_t *__restrict__ osup,
                                                   ull *__restrict__ found) {
    static_assert(TC_OCOL_PAD >= MW, "a window past the last row stays inside the padding");
    __shared__ uint32_t red[BK / TC_WAVE];
    uint32_t all = 0;
    for (int64_t s = (int64_t)blockIdx.x * BK + threadIdx.x; s < m; s += (int64_t)gridDim.x * BK) {
        const int32_t r = orow[s], c = ocol[s];
        int64_t i = s + 1, j = orp[c];
        const int64_t ie = orp[r + 1], je = orp[c + 1];
        uint32_t t = 0;
        while (i < ie && j < je) {
            uint32_t x[MW], y[MW];
#pragma unroll
            for (int e = 0; e < MW; ++e) x[e] = (uint32_t)ocol[i + e];
#pragma unroll
            for (int e = 0; e < MW; ++e) y[e] = (uint32_t)ocol[j + e];
#pragma unroll
            for (int e = 0; e < MW; ++e) {
                x[e] = i + e < ie ? x[e] : 0xFFFFFFFFu;
                y[e] = j + e < je ? y[e] : 0xFFFFFFFEu;
            }
            // every entry up to the smaller of the windows' last ones is
            // settled by this round
            const uint32_t lim = x[MW - 1] < y[MW - 1] ? x[MW - 1] : y[MW - 1];
            uint32_t na = 0, nb = 0;
#pragma unroll
            for (int e = 0; e < MW; ++e) {
                na += x[e] <= lim ? 1u : 0u;
                nb += y[e] <= lim ? 1u : 0u;
            }
            uint32_t hit = 0;
#pragma unroll
            for (int e = 0; e < MW; ++e) {
                uint32_t any = 0;
#pragma unroll
                for (int q = 0; q < MW; ++q) any |= x[e] == y[q] ? 1u << q : 0u;
                if (any) {
                    atomicAdd(&osup[i + e], 1u);
                    atomicAdd(&osup[j + (__ffs((int)any) - 1)], 1u);
                    ++hit;
                }
            }
            t += hit;
            i += na;
            j += nb;
        }
        if (t) atomicAdd(&osup[s], t);
        all += t;
    }
    all = tc_wave_sum(all);
    if (__lane_id() == 0) red[threadIdx.x / TC_WAVE] = all;
    __syncthreads();
    if (threadIdx.x == 0) {
        ull f = 0;
        for (int w = 0; w < BK / TC_WAVE; ++w) f += red[w];
        if (f) atomicAdd(found, f);
    }
}

// SUM 1: the support to canonical order, and acc[r] += Σ sup over r's edges
// (twice the triangles at r).  SUM 2: acc[r] += Σ weight * tri(other end), the
// weight 1 on edges with support and 3 on the others (tri2 holds SUM 1's acc).
template <int SUM>
__global__ __launch_bounds__(BK) void k_slot_sums(int64_t m, int32_t n,
                                                  const int32_t *__restrict__ ocol,
                                                  const int32_t *__restrict__ orow,
                                                  const uint32_t *__restrict__ osup,
                                                  const uint32_t *__restrict__ o2e,
                                                  uint32_t *__restrict__ esup,
                                                  const uint64_t *__restrict__ tri2,
                                                  ull *__restrict__ acc) {
    __shared__ ull top[SLOT_TOP];
    for (int i = threadIdx.x; i < SLOT_TOP; i += BK) top[i] = 0;
    __syncthreads();
    const int32_t base = n > SLOT_TOP ? n - SLOT_TOP : 0;
    const auto add = [&](int32_t r, ull x) {
        if (r >= base) atomicAdd(&top[r - base], x);
        else atomicAdd(&acc[r], x);
    };
    const int64_t step = (int64_t)gridDim.x * BK;
    for (int64_t s0 = (int64_t)blockIdx.x * BK; s0 < m; s0 += step) {
        const int64_t s = s0 + threadIdx.x;
        const bool valid = s < m;
        int32_t r = -1, c = 0;
        ull own = 0, other = 0;
        if (valid) {
            r = orow[s];
            c = ocol[s];
            const uint32_t x = osup[s];
            if constexpr (SUM == 1) {
                esup[o2e[s]] = x;
                own = other = x;
            } else {
                const ull f = x ? 1 : 3;
                own = f * (tri2[c] >> 1);
                other = f * (tri2[r] >> 1);
            }
        }
        bool tail;
        const ull row = run_sum(r, own, tail);
        if (tail && row) add(r, row);
        if (other) add(c, other);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < SLOT_TOP && base + i < n; i += BK)
        if (top[i]) atomicAdd(&acc[base + i], top[i]);
}

// tri in vertex order and its sum per graph (sums).
__global__ __launch_bounds__(BK) void k_slot_tri(int32_t n, const int32_t *__restrict__ rank,
                                                 const uint64_t *__restrict__ tri2,
                                                 const int64_t *__restrict__ vtx_off, int32_t G,
                                                 uint64_t *__restrict__ tri, ull *__restrict__ sums,
                                                 uint32_t *__restrict__ err) {
    __shared__ ull red[BK / TC_WAVE];
    const int64_t per = tc_div_up(tc_div_up(n, gridDim.x), BK) * BK;
    const int64_t a = (int64_t)blockIdx.x * per;
    const int64_t b = a + per < n ? a + per : n;
    ull acc = 0;
    bool odd = false;
    for (int64_t v0 = a; v0 < b; v0 += BK) {
        const int64_t v = v0 + threadIdx.x;
        ull t = 0;
        int32_t g = -1;
        if (v < b) {
            const uint64_t t2 = tri2[rank[v]];
            odd |= (t2 & 1) != 0;
            t = t2 >> 1;
            tri[v] = t;
            if (vtx_off) g = graph_of(vtx_off, G, v);
        }
        if (vtx_off) {
            bool tail;
            const ull x = run_sum(g, t, tail);
            if (tail && x) atomicAdd(&sums[g], x);
        } else {
            acc += t;
        }
    }
    if (odd) atomicOr(err, 2u);
    if (!vtx_off) {
        acc = tc_wave_sum(acc);
        if (__lane_id() == 0) red[threadIdx.x / TC_WAVE] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < BK / TC_WAVE; ++w) acc += red[w];
            if (acc) atomicAdd(&sums[0], acc);
        }
    }
}

// num and tc in vertex order; triG = sums / 3.
__global__ __launch_bounds__(BK) void k_slot_out(int32_t n, const int32_t *__restrict__ rank,
                                                 const ull *__restrict__ acc,
                                                 const uint64_t *__restrict__ tri,
                                                 const ull *__restrict__ sums,
                                                 const int64_t *__restrict__ vtx_off, int32_t G,
                                                 uint64_t *__restrict__ num, double *__restrict__ tcv,
                                                 uint64_t *__restrict__ triG,
                                                 uint32_t *__restrict__ err) {
    const int64_t t0 = (int64_t)blockIdx.x * BK + threadIdx.x, step = (int64_t)gridDim.x * BK;
    for (int64_t g = t0; g < G; g += step) {
        const ull s = sums[g];
        if (s % 3) atomicOr(err, 4u);
        const ull t = s / 3;
        if (t > ~0ull / 3) atomicOr(err, 8u);
        triG[g] = t;
    }
    for (int64_t v = t0; v < n; v += step) {
        const uint64_t x = acc[rank[v]] + tri[v];
        num[v] = x;
        // one correctly rounded binary64 division, as in the other forms
        const ull tg = sums[vtx_off ? graph_of(vtx_off, G, v) : 0] / 3;
        tcv[v] = tg == 0 ? 0.0 : __ddiv_rn((double)x, (double)(3 * tg));
    }
}

}  // namespace

tc_status tc_count_slots(tc_graph *g, unsigned long long *found, hipStream_t s) {
    k_slot_count<<<grid_for(g->m, 4096), BK, 0, s>>>(g->m, g->orp, g->ocol, g->orow, g->osup, found);
    TC_LAUNCHED();
    return TC_OK;
}

tc_status tc_aggregate_slots(tc_graph *g, hipStream_t s) {
    const int32_t n = g->n, G = g->num_graphs;
    const int64_t m = g->m;
    if (!g->esup) TC_TRY(tc_graph_alloc(g, &g->esup, m, s));
    if (!g->tri) TC_TRY(tc_graph_alloc(g, &g->tri, n, s));
    if (!g->num) TC_TRY(tc_graph_alloc(g, &g->num, n, s));
    if (!g->tcv) TC_TRY(tc_graph_alloc(g, &g->tcv, n, s));
    const int64_t *voff = G > 1 ? g->vtx_off : nullptr;
    tc_scratch tmp(s);
    ull *acc = nullptr;  // twice the triangles by rank, the numerators by rank, sums
    TC_TRY(tmp.get(&acc, 2 * (int64_t)n + G));
    ull *num2 = acc + n, *sums = num2 + n;
    TC_HIP(hipMemsetAsync(acc, 0, sizeof(ull) * (2 * (int64_t)n + G), s));
    k_slot_sums<1><<<grid_for(m, SUM_BLOCKS), BK, 0, s>>>(m, n, g->ocol, g->orow, g->osup, g->o2e,
                                                         g->esup, nullptr, acc);
    TC_LAUNCHED();
    const uint64_t *tri2 = reinterpret_cast<const uint64_t *>(acc);
    k_slot_tri<<<grid_for(n, SUM_BLOCKS), BK, 0, s>>>(n, g->rank, tri2, voff, G, g->tri, sums, g->err);
    TC_LAUNCHED();
    tc_prof_mark(g, 10, s);
    k_slot_sums<2><<<grid_for(m, SUM_BLOCKS), BK, 0, s>>>(m, n, g->ocol, g->orow, g->osup, nullptr,
                                                         nullptr, tri2, num2);
    TC_LAUNCHED();
    k_slot_out<<<grid_for(n > G ? n : G, 65536), BK, 0, s>>>(n, g->rank, num2, g->tri, sums, voff, G,
                                                            g->num, g->tcv, g->triG, g->err);
    TC_LAUNCHED();
    tc_prof_mark(g, 11, s);
    return TC_OK;
}
