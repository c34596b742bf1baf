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
// What bounds it: the merge is bound by its comparisons (46% of the VALU's time,
// the lanes' rounds differing) and the random rows N_H(c), the sums by the
// atomics on the higher ends, so each workgroup sums what it can in LDS and adds
// it once at its end; a hub then costs one atomic per workgroup and not one per
// edge (11 ns each on one word).
//
// Whole calls, from the middle pivot with its transposition sort, bit matrices
// and rank-space sums to this: 5 M uniform pairs over 1.25 M vertices 2593 to
// 1221 us, 512 BA graphs with 17.8 M edges 8774 to 3401 us (count 613 us, sums
// 175 and 148 us).
#include "tc_internal.h"

namespace {

constexpr int BK = 256;
constexpr int MW = 8;  // entries of each list per round of the merge
constexpr int COUNT_RUN = 2048;       // slots per workgroup of the count, at most
constexpr int SUM_BLOCK = 1024;
constexpr int SUM_WIN = 8192;         // ranks summed in LDS: 64 KB, two workgroups per CU
// Workgroups of the sums.  One graph: all resident, as each adds its LDS words
// once (BA graph of 8 M edges: 64 us against 77 with 4096).  Many graphs: short
// runs, so that the graphs in flight on an XCD fit its L2 (17.8 M edges in 512
// graphs: 175 us against 371 with 512, for the scattered supports).
constexpr int64_t SUM_RUNS = 512, SUM_RUNS_GRAPHS = 4096;
constexpr unsigned SUM_BLOCKS = 1024;
using ull = unsigned long long;

static inline unsigned grid_for(int64_t n, unsigned most) {
    const int64_t g = tc_div_up(n, BK);
    return (unsigned)(g < 1 ? 1 : (g < most ? g : most));
}

// First slot of this workgroup's run.  Workgroups go to the 8 XCDs in turn.  With
// many graphs each XCD takes an eighth of the runs in order, so that its L2 holds
// the graphs that its workgroups read (gridDim.x is a multiple of 8); one graph's
// runs are dealt out, as the last ones, of the highest ranks, have the most work.
__device__ __forceinline__ int64_t first_slot(int64_t run, bool graphs) {
    const int64_t b = blockIdx.x;
    return (graphs ? (b % 8) * (gridDim.x / 8) + b / 8 : b) * run;
}

// Slots per workgroup for `most` workgroups, a multiple of block; the grid.
static inline int64_t run_for(int64_t m, int64_t most, int64_t block) {
    return tc_div_up(tc_div_up(m, most), block) * block;
}
static inline unsigned runs_grid(int64_t m, int64_t run) {
    return (unsigned)(tc_div_up(tc_div_up(m, run), 8) * 8);
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
// loaded whole.
// A workgroup takes a run of slots, whose rows it keeps in LDS with their
// counters: half of the merge's reads and of its adds stay there (17.8 M edges
// in 512 graphs: 824 to 613 us, a BA graph of 7.5 M edges: 227 to 199).  The
// last row may go on past the run, by less than a row.
__global__ __launch_bounds__(BK) void k_slot_count(int64_t m, int32_t run, bool graphs,
                                                   const int64_t *__restrict__ orp,
                                                   const int32_t *__restrict__ ocol,
                                                   const int32_t *__restrict__ orow,
                                                   uint32_t *__restrict__ osup,
                                                   ull *__restrict__ found) {
    static_assert(TC_OCOL_PAD >= MW, "a window past the last row stays inside the padding");
    __shared__ uint32_t red[BK / TC_WAVE];
    __shared__ uint32_t row[COUNT_RUN + TC_SLOTS_MAX_DPLUS + MW];
    __shared__ uint32_t sup[COUNT_RUN + TC_SLOTS_MAX_DPLUS];
    const int64_t first = first_slot(run, graphs);
    if (first >= m) return;
    const int len = (int)(first + run < m ? run : m - first);
    // the run and what its last row may have after it
    const int all_len = (int)(first + len + TC_SLOTS_MAX_DPLUS < m ? len + TC_SLOTS_MAX_DPLUS : m - first);
    for (int i = threadIdx.x; i < all_len; i += BK) {
        row[i] = (uint32_t)ocol[first + i];
        sup[i] = 0;
    }
    __syncthreads();
    uint32_t all = 0;
    for (int s = threadIdx.x; s < len; s += BK) {
        const int32_t r = orow[first + s], c = (int32_t)row[s];
        int64_t j = orp[c];
        const int64_t je = orp[c + 1];
        int i = s + 1;
        const int ie = (int)(orp[r + 1] - first);
        uint32_t t = 0;
        while (i < ie && j < je) {
            uint32_t x[MW], y[MW];
#pragma unroll
            for (int e = 0; e < MW; ++e) y[e] = (uint32_t)ocol[j + e];
#pragma unroll
            for (int e = 0; e < MW; ++e) x[e] = row[i + e];
            // entries past a list's end: values that equal nothing
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
#pragma unroll
            for (int e = 0; e < MW; ++e) {
                uint32_t any = 0;
#pragma unroll
                for (int q = 0; q < MW; ++q) any |= x[e] == y[q] ? 1u << q : 0u;
                if (any) {
                    atomicAdd(&sup[i + e], 1u);
                    atomicAdd(&osup[j + (__ffs((int)any) - 1)], 1u);
                    ++t;
                }
            }
            i += na;
            j += nb;
        }
        if (t) atomicAdd(&sup[s], t);
        all += t;
    }
    all = tc_wave_sum(all);
    if (__lane_id() == 0) red[threadIdx.x / TC_WAVE] = all;
    __syncthreads();
    for (int i = threadIdx.x; i < all_len; i += BK)
        if (sup[i]) atomicAdd(&osup[first + i], sup[i]);
    if (threadIdx.x == 0) {
        ull f = 0;
        for (int w = 0; w < BK / TC_WAVE; ++w) f += red[w];
        if (f) atomicAdd(found, f);
    }
}

// SUM 1: the support to canonical order, and acc[r] += Σ sup over r's edges
// (twice the triangles at r).  SUM 2: acc[r] += Σ weight * tri(other end), the
// weight 1 on edges with support and 3 on the others (tri2 holds SUM 1's acc).
//
// A workgroup takes a run of slots.  Its rows and their higher ends lie between
// the first row and the last vertex of the last row's graph; the SUM_WIN highest
// ranks of that span are summed in LDS and added once.
template <int SUM>
__global__ __launch_bounds__(SUM_BLOCK) void k_slot_sums(int64_t m, int64_t run, int32_t n,
                                                         const int32_t *__restrict__ ocol,
                                                         const int32_t *__restrict__ orow,
                                                         const uint32_t *__restrict__ osup,
                                                         const uint32_t *__restrict__ o2e,
                                                         uint32_t *__restrict__ esup,
                                                         const uint64_t *__restrict__ tri2,
                                                         const int64_t *__restrict__ vtx_off, int32_t G,
                                                         ull *__restrict__ acc) {
    __shared__ ull win[SUM_WIN];
    __shared__ int32_t span[2];
    const int64_t a = first_slot(run, vtx_off != nullptr);
    const int64_t b = a + run < m ? a + run : m;
    if (a >= b) return;
    if (threadIdx.x == 0) {
        const int32_t r = orow[a];
        const int32_t e = vtx_off ? (int32_t)vtx_off[tc_graph_of(vtx_off, G, orow[b - 1]) + 1] : n;
        span[0] = e - SUM_WIN > r ? e - SUM_WIN : r;
        span[1] = e;
    }
    __syncthreads();
    const int32_t base = span[0], len = span[1] - base;  // at most SUM_WIN
    for (int i = threadIdx.x; i < len; i += SUM_BLOCK) win[i] = 0;
    __syncthreads();
    const auto add = [&](int32_t r, ull x) {
        if ((uint32_t)(r - base) < (uint32_t)len) atomicAdd(&win[r - base], x);
        else atomicAdd(&acc[r], x);
    };
    for (int64_t s0 = a; s0 < b; s0 += SUM_BLOCK) {
        const int64_t s = s0 + threadIdx.x;
        const bool valid = s < b;
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
    for (int i = threadIdx.x; i < len; i += SUM_BLOCK)
        if (win[i]) atomicAdd(&acc[base + i], win[i]);
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
            if (vtx_off) g = tc_graph_of(vtx_off, G, v);
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
        const ull tg = sums[vtx_off ? tc_graph_of(vtx_off, G, v) : 0] / 3;
        tcv[v] = tg == 0 ? 0.0 : __ddiv_rn((double)x, (double)(3 * tg));
    }
}

}  // namespace

tc_status tc_count_slots(tc_graph *g, unsigned long long *found, hipStream_t s) {
    const int64_t most = run_for(g->m, 4096, BK), run = most < COUNT_RUN ? most : COUNT_RUN;
    k_slot_count<<<runs_grid(g->m, run), BK, 0, s>>>(g->m, (int32_t)run, g->rank_by_graph, g->orp, g->ocol, g->orow, g->osup, found);
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
    // twice the triangles by rank, in num until that is written at the end; the
    // numerators by rank, sums
    ull *acc = reinterpret_cast<ull *>(g->num), *num2 = nullptr;
    TC_TRY(tmp.get(&num2, (int64_t)n + G));
    ull *sums = num2 + n;
    TC_TRY(tc_zero({{acc, 2 * (int64_t)n}, {num2, 2 * ((int64_t)n + G)}}, s));
    const int64_t run = run_for(m, g->rank_by_graph ? SUM_RUNS_GRAPHS : SUM_RUNS, SUM_BLOCK);
    const int64_t *span = g->rank_by_graph ? voff : nullptr;
    k_slot_sums<1><<<runs_grid(m, run), SUM_BLOCK, 0, s>>>(m, run, n, g->ocol, g->orow, g->osup, g->o2e,
                                                          g->esup, nullptr, span, G, acc);
    TC_LAUNCHED();
    const uint64_t *tri2 = reinterpret_cast<const uint64_t *>(acc);
    k_slot_tri<<<grid_for(n, SUM_BLOCKS), BK, 0, s>>>(n, g->rank, tri2, voff, G, g->tri, sums, g->err);
    TC_LAUNCHED();
    tc_prof_mark(g, 10, s);
    k_slot_sums<2><<<runs_grid(m, run), SUM_BLOCK, 0, s>>>(m, run, n, g->ocol, g->orow, g->osup, nullptr,
                                                          nullptr, tri2, span, G, num2);
    TC_LAUNCHED();
    k_slot_out<<<grid_for(n > G ? n : G, 65536), BK, 0, s>>>(n, g->rank, num2, g->tri, sums, voff, G,
                                                            g->num, g->tcv, g->triG, g->err);
    TC_LAUNCHED();
    tc_prof_mark(g, 11, s);
    return TC_OK;
}
