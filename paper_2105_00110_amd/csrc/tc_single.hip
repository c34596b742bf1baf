// Build and count of one small graph by one workgroup each (tc_small.h).
//
// A graph of at most 16384 pairs over at most 4096 vertices: one launch builds
// everything that the general path builds with some thirty (canonical edges,
// degrees, degree order, oriented rows), and one launch counts and aggregates.
// What bounds such a call is launches and waits, not work: an ER graph of 10 k
// pairs took 311 us a call by the general path, 142 us so (build 61 us, count
// 32 us of device time).  Larger graphs gain more from all compute units than
// they lose in launches.
#include "tc_internal.h"
#include "tc_small.h"

namespace {

using namespace tc_small;
constexpr int BLOCK = 1024;
using L1024 = Lds<BLOCK>;

struct BuildOut {
    int32_t *eu, *ev;
    uint32_t *run_us;
    int64_t *row_ptr;
    int32_t *rank, *perm;
    int64_t *orp;
    int32_t *ocol;
    uint32_t *o2e;
    int32_t *orow;
    uint32_t *err;   // error bits, largest degree
    uint32_t *info;  // edges, id out of range, longest row, largest degree
};

__global__ __launch_bounds__(BLOCK) void k_single_build(const int32_t *__restrict__ src,
                                                        const int32_t *__restrict__ dst, uint32_t P,
                                                        uint32_t n, BuildOut o) {
    __shared__ L1024 L;
    const int tid = threadIdx.x;
    const int b = bits_of(n > 1 ? n - 1 : 1);
    const int itn = (int)((P + BLOCK - 1) / BLOCK);
    const uint32_t none = (uint32_t)((1ull << (2 * b)) - 1ull);
    uint32_t key[ITEMS];
    bool bad = false;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        key[it] = none;
        if (it < itn) {
            const uint32_t i = elem(it, itn);
            if (i < P) {
                const uint32_t x = (uint32_t)src[i], y = (uint32_t)dst[i];
                if (x >= n || y >= n) bad = true;
                else if (x != y) key[it] = x < y ? x << b | y : y << b | x;
            }
        }
    }
    bad = __builtin_amdgcn_readfirstlane(__syncthreads_or(bad)) != 0;
    if (tid == 0) {
        o.err[0] = o.err[1] = o.err[2] = o.err[3] = 0;
        o.info[1] = bad ? 1u : 0u;
    }
    if (bad) return;
    Edges E;
    const uint32_t m = canonical<BLOCK>(key, itn, b, E, L);
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        if (E.ends[it] != NONE) {
            const uint32_t lo = E.ends[it] >> 16, e = E.tag[it], i = elem(it, itn);
            o.eu[e] = (int32_t)lo;
            o.ev[e] = (int32_t)(E.ends[it] & 0xFFFFu);
            if (i == 0 || L.xchg[i - 1] >> b != lo) o.run_us[lo] = e;  // first of its end's run
        }
    __syncthreads();
    const uint32_t dmax = degree_rank<BLOCK>(E, n, L, [&](uint32_t r, uint32_t v) {
        o.perm[r] = (int32_t)v;
        o.rank[v] = (int32_t)r;
    });
    // row offsets of the symmetric adjacency: consecutive vertices per thread
    {
        constexpr int PER = L1024::NMAX / BLOCK;
        uint32_t d[PER], sum = 0, all;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t v = tid * PER + k;
            d[k] = v < n ? L.cnt[v] : 0u;
            sum += d[k];
        }
        uint32_t at = wg_scan<BLOCK>(sum, &all, L.wsum);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t v = tid * PER + k;
            if (v < n) o.row_ptr[v] = at;
            at += d[k];
        }
        if (tid == 0) o.row_ptr[n] = all;
    }
    const uint32_t longest = orient<BLOCK>(E, n, m, L);
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        if (E.ends[it] != NONE) {
            const uint32_t s = E.tag[it] >> 16;
            o.ocol[s] = (int32_t)(E.ends[it] & 0xFFFFu);
            o.orow[s] = (int32_t)(E.ends[it] >> 16);
            o.o2e[s] = E.tag[it] & 0xFFFFu;
        }
    for (uint32_t r = tid; r <= n; r += BLOCK) o.orp[r] = L.orp[r];
    if (tid == 0) {
        o.info[0] = m;
        o.info[2] = longest;
        o.info[3] = dmax;
        o.err[1] = dmax;
    }
}

struct CountArgs {
    const int64_t *orp;
    const int32_t *ocol, *orow, *rank;
    const uint32_t *o2e;
    uint32_t *osup, *esup;
    uint64_t *tri, *num;
    double *tcv;
    uint64_t *triG;  // [2]: triangles, and again as the count's own total
    uint32_t *err;
};

__global__ __launch_bounds__(BLOCK) void k_single_count(uint32_t m, uint32_t n, CountArgs a) {
    __shared__ L1024 L;
    const int tid = threadIdx.x;
    for (uint32_t s = tid; s < m; s += BLOCK) L.xchg[s] = (uint32_t)a.orow[s] << 16 | (uint32_t)a.ocol[s];
    for (uint32_t r = tid; r <= n; r += BLOCK) L.orp[r] = (uint16_t)a.orp[r];
    count_slots<BLOCK>(m, n, L);
    for (uint32_t s = tid; s < m; s += BLOCK) {
        const uint32_t x = support(s, L);
        a.osup[s] = x;
        a.esup[a.o2e[s]] = x;
    }
    const uint32_t three_t = slot_sums<BLOCK>(m, L);
    const uint64_t tg = three_t / 3;
    bool odd = false;
    for (uint32_t v = tid; v < n; v += BLOCK) {
        const uint32_t r = (uint32_t)a.rank[v];
        odd |= (L.tri[r] & 1u) != 0;
        const uint64_t t = L.tri[r] >> 1, x = L.num[r] + t;
        a.tri[v] = t;
        a.num[v] = x;
        // one correctly rounded binary64 division, as in the other forms
        a.tcv[v] = tg == 0 ? 0.0 : __ddiv_rn((double)x, (double)(3 * tg));
    }
    if (odd) atomicOr(a.err, 2u);
    if (tid == 0) {
        if (three_t % 3) atomicOr(a.err, 4u);
        a.triG[0] = a.triG[1] = tg;
    }
}

}  // namespace

bool tc_single_fits(int64_t P, int32_t n) {
    return P > 0 && P <= L1024::CAP && n > 0 && n <= L1024::NMAX;
}

tc_status tc_single_build(tc_graph *g, const int32_t *d_src, const int32_t *d_dst, int64_t P,
                          hipStream_t s) {
    const int32_t n = g->n;
    tc_scratch tmp(s);
    BuildOut o;
    // the edge arrays take the pair count: the edges are counted by the launch
    TC_TRY(tc_graph_alloc(g, &g->err, 4, s));
    TC_TRY(tc_graph_alloc(g, &g->eu, P, s));
    TC_TRY(tc_graph_alloc(g, &g->ev, P, s));
    TC_TRY(tc_graph_alloc(g, &g->run_us, n, s));
    TC_TRY(tc_graph_alloc(g, &g->row_ptr, (int64_t)n + 1, s));
    TC_TRY(tc_graph_alloc(g, &g->rank, n, s));
    TC_TRY(tc_graph_alloc(g, &g->perm, n, s));
    TC_TRY(tc_graph_alloc(g, &g->orp, (int64_t)n + 1, s));
    TC_TRY(tc_graph_alloc(g, &g->ocol, P + TC_OCOL_PAD, s));
    TC_TRY(tc_graph_alloc(g, &g->o2e, P, s));
    TC_TRY(tc_graph_alloc(g, &g->orow, P, s));
    TC_TRY(tmp.get(&o.info, 4));
    o.eu = g->eu;
    o.ev = g->ev;
    o.run_us = g->run_us;
    o.row_ptr = g->row_ptr;
    o.rank = g->rank;
    o.perm = g->perm;
    o.orp = g->orp;
    o.ocol = g->ocol;
    o.o2e = g->o2e;
    o.orow = g->orow;
    o.err = g->err;
    k_single_build<<<1, BLOCK, 0, s>>>(d_src, d_dst, (uint32_t)P, (uint32_t)n, o);
    TC_LAUNCHED();
    for (int k = 1; k <= 3; ++k) tc_prof_mark(g, k, s);
    uint32_t info[4] = {0, 0, 0, 0};
    TC_TRY(tc_read({{info, o.info, 4}}, s));
    if (info[1]) return TC_ERR_VERTEX_RANGE;
    g->m = info[0];
    g->max_dplus = (int32_t)info[2];
    g->max_degree = (int32_t)info[3];
    g->single = true;
    return TC_OK;
}

tc_status tc_single_count(tc_graph *g, hipStream_t s) {
    const int32_t n = g->n;
    if (!g->esup) TC_TRY(tc_graph_alloc(g, &g->esup, g->m, s));
    if (!g->tri) TC_TRY(tc_graph_alloc(g, &g->tri, n, s));
    if (!g->num) TC_TRY(tc_graph_alloc(g, &g->num, n, s));
    if (!g->tcv) TC_TRY(tc_graph_alloc(g, &g->tcv, n, s));
    const CountArgs a{g->orp,  g->ocol, g->orow, g->rank, g->o2e,  g->osup,
                      g->esup, g->tri,  g->num,  g->tcv,  g->triG, g->err};
    k_single_count<<<1, BLOCK, 0, s>>>((uint32_t)g->m, (uint32_t)n, a);
    TC_LAUNCHED();
    return TC_OK;
}
