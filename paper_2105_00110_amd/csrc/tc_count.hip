// Triangle counting with per-edge support on the degree-ordered orientation.
//
// In rank space every triangle is v < u < w with u, w ∈ N_H(v) and
// w ∈ N_H(u); it is found exactly once, from row v, while intersecting
// N_H(v) with N_H(u) (the appendix's alternative TriangleNeighbor
// procedure: only the low and middle vertices' higher-ordered sets are
// intersected, only the high vertex is ever returned).  For each common w
// at index l of N_H(v) and index r of N_H(u), the procedure marks L_v(l)
// and L_u(r), and marks L_v(i) for u's own index i if anything was found;
// here each mark is a count instead, so the slot ends holding the number
// of triangles on its edge (the value of T = A² ∘ A there):
//     sup(v,w) += 1,   sup(u,w) += 1,   sup(v,u) += |N_H(v) ∩ N_H(u)|.
//
// MI355X mapping.  Row v's set N_H(v) is put into an LDS hash table (key =
// rank, value = index in the row); the wavefront streams N_H(u) for each u
// of the row with coalesced 64-wide loads and probes the table, so the
// candidate stream is Σ_{u ∈ N_H(v)} |N_H(u)| reads.  sup(v,·) accumulates
// in LDS and is flushed once per slot; sup(u,w) is one global atomic per
// triangle; sup(v,u) is a ballot/popcount reduction.  Streaming of N_H(u)
// stops at the first entry above max N_H(v), since both lists are sorted.
//
// Rows are binned by d+ = |N_H(v)|: rows with d+ < 2 close no triangle;
// "light" rows (d+ <= light_max_dplus) get one wavefront each; "heavy"
// rows a workgroup sharing one table; "huge" rows (table larger than the
// LDS budget) probe by binary search in device memory.  The schedule never
// changes a result: every count is an integer sum.
#include "tc_internal.h"
#include "tc_table.h"

namespace {

constexpr int BK = 256;
constexpr int UNROLL = 4;  // independent candidate loads in flight per lane
// Above the slot merge TC_ALGO_AUTO takes the middle pivot from this many
// edges (whole calls, low / middle, us: R-MAT scale 13, 183 k edges 852 / 661, scale
// 14, 213 k 871 / 736 and 389 k 1060 / 744, scale 15, 441 k 902 / 686; K_660, 217 k
// 1605 / 811, K_1000 2003 / 1099; half of all pairs of 1000 vertices, 250 k 1435 /
// 646; a tenth of those of 3000, 450 k 1040 / 664; BA attach 150, 441 k 842 / 603).
constexpr int64_t AUTO_MID_MIN_EDGES = 200000;
using namespace tc_tab;

static inline unsigned grid_for(int64_t n, int block = BK) {
    int64_t g = tc_div_up(n, block);
    if (g < 1) g = 1;
    if (g > 0x7FFFFFFF) g = 0x7FFFFFFF;
    return (unsigned)g;
}

// Streams N_H(u) = ocol[ub, ue) against row v and applies the support
// updates; returns |N_H(v) ∩ N_H(u)| (wave-uniform).  Each lane keeps
// UNROLL loads in flight; the stream stops once it passes vmax = max N_H(v).
template <bool GLOBAL_LOOKUP>
__device__ __forceinline__ uint32_t stream_u(const int32_t *__restrict__ ocol, int64_t ub,
                                             int64_t ue, uint32_t vmax, const RowTable &t,
                                             uint32_t *lsup, int64_t vstart, int dv,
                                             uint32_t *__restrict__ osup) {
    const int lane = __lane_id();
    uint32_t c = 0;
    for (int64_t jb = ub; jb < ue; jb += TC_WAVE * UNROLL) {
        uint32_t w[UNROLL];
#pragma unroll
        for (int q = 0; q < UNROLL; ++q) {
            const int64_t j = jb + q * TC_WAVE + lane;
            w[q] = j < ue ? (uint32_t)ocol[j] : EMPTY;
        }
        // lane 0's first load is the smallest candidate of the chunk
        if ((uint32_t)__shfl(w[0], 0, TC_WAVE) > vmax) break;
        // EMPTY (past the row end) is above every rank: never looked up
        int pq[UNROLL];
        if constexpr (GLOBAL_LOOKUP) {
#pragma unroll
            for (int q = 0; q < UNROLL; ++q)
                pq[q] = w[q] <= vmax ? row_search(ocol, vstart, dv, w[q]) : -1;
        } else {
            table_find_n<UNROLL>(t, w, vmax, pq);
        }
#pragma unroll
        for (int q = 0; q < UNROLL; ++q) {
            const int p = pq[q];
            const bool hit = p >= 0;
            if (hit) {
                if constexpr (GLOBAL_LOOKUP) atomicAdd(&osup[vstart + p], 1u);
                else atomicAdd(&lsup[p], 1u);
                atomicAdd(&osup[jb + q * TC_WAVE + lane], 1u);
            }
            c += (uint32_t)__popcll(__ballot(hit));
        }
        if ((uint32_t)__shfl(w[UNROLL - 1], TC_WAVE - 1, TC_WAVE) > vmax) break;
    }
    return c;
}

// Per-wave LDS footprint of the light kernel (bytes, 16-aligned).
__host__ __device__ __forceinline__ size_t light_wave_bytes(int dcap) {
    const size_t nb = (size_t)1 << bucket_bits(dcap);
    return (16 * nb + 2 * 4 * nb + 4 * (size_t)dcap + 15) & ~(size_t)15;
}

// One wavefront per light row.
__global__ __launch_bounds__(1024) void k_count_light(const int64_t *__restrict__ orp,
                                                      const int32_t *__restrict__ ocol,
                                                      const int32_t *__restrict__ rows,
                                                      const uint32_t *__restrict__ row_count,
                                                      int dcap,
                                                      uint32_t *__restrict__ osup,
                                                      unsigned long long *__restrict__ tri_total) {
    extern __shared__ uint4 lds4[];
    const int wpb = blockDim.x / TC_WAVE;
    const int wv = threadIdx.x / TC_WAVE;
    const int lane = __lane_id();
    const int nbmax = 1 << bucket_bits(dcap);
    char *base = reinterpret_cast<char *>(lds4) + (size_t)wv * light_wave_bytes(dcap);
    uint32_t *keys = reinterpret_cast<uint32_t *>(base);
    uint16_t *pos = reinterpret_cast<uint16_t *>(base + 16 * (size_t)nbmax);
    uint32_t *lsup = reinterpret_cast<uint32_t *>(base + 24 * (size_t)nbmax);
    unsigned long long found = 0;
    const int64_t nrows = *row_count;
    for (int64_t ri = (int64_t)blockIdx.x * wpb + wv; ri < nrows; ri += (int64_t)gridDim.x * wpb) {
        const int32_t r = rows[ri];
        const int64_t start = orp[r];
        const int d = (int)(orp[r + 1] - start);
        const RowTable t{keys, pos, bucket_bits(d)};
        for (int j = lane; j < (4 << t.bb); j += TC_WAVE) keys[j] = EMPTY;
        for (int j = lane; j < d; j += TC_WAVE) lsup[j] = 0;
        for (int j = lane; j < d; j += TC_WAVE) table_insert(t, (uint32_t)ocol[start + j], j);
        const uint32_t vmax = (uint32_t)ocol[start + d - 1];
        for (int i0 = 0; i0 < d - 1; i0 += TC_WAVE) {
            const int ii = i0 + lane;
            int64_t ub_l = 0, ue_l = 0;
            if (ii < d - 1) {
                const int32_t u = ocol[start + ii];
                ub_l = orp[u];
                ue_l = orp[u + 1];
            }
            const int cnt = min(TC_WAVE, d - 1 - i0);
            for (int k = 0; k < cnt; ++k) {
                const int64_t ub = __shfl(ub_l, k, TC_WAVE), ue = __shfl(ue_l, k, TC_WAVE);
                const uint32_t c = stream_u<false>(ocol, ub, ue, vmax, t, lsup, start, d, osup);
                if (c != 0 && lane == 0) atomicAdd(&lsup[i0 + k], c);
                found += c;
            }
        }
        for (int j = lane; j < d; j += TC_WAVE) {
            const uint32_t x = lsup[j];
            if (x) atomicAdd(&osup[start + j], x);
        }
    }
    if (lane == 0 && found) atomicAdd(tri_total, found);
}

// LDS footprint of the heavy kernel for rows of at most dmax entries.
static inline size_t heavy_bytes(int dmax) {
    const size_t nb = (size_t)1 << bucket_bits(dmax);
    return 16 * nb + 8 * nb + 4 * (size_t)dmax;
}

// One workgroup per heavy row (GLOBAL_LOOKUP: no table, binary search in
// device memory, for rows whose table would not fit).  Wavefront wv takes
// the row's u at indices wv, wv + wpb, wv + 2·wpb, ...
template <bool GLOBAL_LOOKUP>
__global__ __launch_bounds__(1024) void k_count_heavy(const int64_t *__restrict__ orp,
                                                      const int32_t *__restrict__ ocol,
                                                      const int32_t *__restrict__ rows,
                                                      const uint32_t *__restrict__ row_count,
                                                      int dmax,
                                                      uint32_t *__restrict__ osup,
                                                      unsigned long long *__restrict__ tri_total) {
    extern __shared__ uint4 lds4[];
    const int wpb = blockDim.x / TC_WAVE;
    const int wv = threadIdx.x / TC_WAVE;
    const int lane = __lane_id();
    const int nbmax = GLOBAL_LOOKUP ? 0 : (1 << bucket_bits(dmax));
    char *base = reinterpret_cast<char *>(lds4);
    uint32_t *keys = reinterpret_cast<uint32_t *>(base);
    uint16_t *pos = reinterpret_cast<uint16_t *>(base + 16 * (size_t)nbmax);
    uint32_t *lsup = reinterpret_cast<uint32_t *>(base + 24 * (size_t)nbmax);
    unsigned long long found = 0;
    const int64_t nrows = *row_count;
    for (int64_t bi = blockIdx.x; bi < nrows; bi += gridDim.x) {
        const int32_t r = rows[bi];
        const int64_t start = orp[r];
        const int d = (int)(orp[r + 1] - start);
        RowTable t{keys, pos, 0};
        if constexpr (!GLOBAL_LOOKUP) {
            t.bb = bucket_bits(d);
            for (int j = threadIdx.x; j < (4 << t.bb); j += blockDim.x) keys[j] = EMPTY;
            for (int j = threadIdx.x; j < d; j += blockDim.x) lsup[j] = 0;
            __syncthreads();
            for (int j = threadIdx.x; j < d; j += blockDim.x)
                table_insert(t, (uint32_t)ocol[start + j], j);
            __syncthreads();
        }
        const uint32_t vmax = (uint32_t)ocol[start + d - 1];
        const int nu = d - 1;  // the last entry closes no triangle in this row
        for (int k0 = 0; wv + wpb * k0 < nu; k0 += TC_WAVE) {
            const int ii = wv + wpb * (k0 + lane);
            int64_t ub_l = 0, ue_l = 0;
            if (ii < nu) {
                const int32_t u = ocol[start + ii];
                ub_l = orp[u];
                ue_l = orp[u + 1];
            }
            for (int k = 0; k < TC_WAVE; ++k) {
                const int i = wv + wpb * (k0 + k);
                if (i >= nu) break;
                const int64_t ub = __shfl(ub_l, k, TC_WAVE), ue = __shfl(ue_l, k, TC_WAVE);
                const uint32_t c =
                    stream_u<GLOBAL_LOOKUP>(ocol, ub, ue, vmax, t, lsup, start, d, osup);
                if (c != 0 && lane == 0) {
                    if constexpr (GLOBAL_LOOKUP) atomicAdd(&osup[start + i], c);
                    else atomicAdd(&lsup[i], c);
                }
                found += c;
            }
        }
        if constexpr (!GLOBAL_LOOKUP) {
            __syncthreads();
            for (int j = threadIdx.x; j < d; j += blockDim.x) {
                const uint32_t x = lsup[j];
                if (x) atomicAdd(&osup[start + j], x);
            }
            __syncthreads();
        }
    }
    if (lane == 0 && found) atomicAdd(tri_total, found);
}

// The rows of each bin (2 <= d+ <= light_max, then below huge_min, then the
// others), in any order; cnt[0..2] their numbers.  The count kernels read the
// numbers on the device, so nothing waits for them (flags, a scan and a write
// for each bin and a read-back were 13 launches and a wait).
constexpr int BR_TILE = 2048;

__global__ __launch_bounds__(BK) void k_bin_rows(int32_t n, const int64_t *__restrict__ orp,
                                                 int light_max, int huge_min,
                                                 int32_t *__restrict__ light,
                                                 int32_t *__restrict__ heavy,
                                                 int32_t *__restrict__ huge,
                                                 uint32_t *__restrict__ cnt) {
    constexpr int PER = BR_TILE / BK;
    __shared__ uint32_t lds[BK / TC_WAVE + 1];
    const int64_t base = (int64_t)blockIdx.x * BR_TILE;
    int bin[PER];
    uint32_t c[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t r = base + k * BK + threadIdx.x;
        const int64_t d = r < n ? orp[r + 1] - orp[r] : 0;
        bin[k] = d < 2 ? -1 : (d <= light_max ? 0 : (d < huge_min ? 1 : 2));
#pragma unroll
        for (int q = 0; q < 3; ++q) c[q] += bin[k] == q ? 1u : 0u;
    }
    uint32_t p0 = tc_block_reserve<BK>(c[0], &cnt[0], lds), p1 = 0, p2 = 0;
    if (__syncthreads_or(c[1] | c[2])) {
        p1 = tc_block_reserve<BK>(c[1], &cnt[1], lds);
        p2 = tc_block_reserve<BK>(c[2], &cnt[2], lds);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int32_t r = (int32_t)(base + k * BK + threadIdx.x);
        if (bin[k] == 0) light[p0++] = r;
        else if (bin[k] == 1) heavy[p1++] = r;
        else if (bin[k] == 2) huge[p2++] = r;
    }
}

}  // namespace

tc_status tc_tuning_default(tc_tuning *t) {
    if (!t) return TC_ERR_INVALID_ARG;
    t->light_max_dplus = 512;
    t->heavy_block = 256;
    t->light_block = 256;
    t->lds_max_entries = 4096;
    t->algorithm = TC_ALGO_AUTO;
    t->item_pairs = 512;
    t->bitmap_words = 4096;
    t->light_bitmap_pairs = TC_LIGHT_BITMAP_PAIRS;
    return TC_OK;
}

static bool tuning_valid(const tc_tuning *t) {
    auto pow2 = [](int x) { return x > 0 && (x & (x - 1)) == 0; };
    return t->light_max_dplus >= 2 && t->light_max_dplus <= 1024 && t->heavy_block >= 64 &&
           t->heavy_block <= 1024 && t->heavy_block % 64 == 0 && t->light_block >= 64 &&
           t->light_block <= 1024 && t->light_block % 64 == 0 && pow2(t->lds_max_entries) &&
           t->lds_max_entries >= 1024 && t->lds_max_entries <= 16384 && t->algorithm >= 0 &&
           t->algorithm <= 2 && t->item_pairs >= 64 && t->item_pairs <= 65536 &&
           t->item_pairs % 64 == 0 &&
           (t->bitmap_words == 0 ||
            (pow2(t->bitmap_words) && t->bitmap_words >= 256 && t->bitmap_words <= 8192)) &&
           t->light_bitmap_pairs >= 0;
}

// The forms that AUTO chooses between.
enum class Form { SLOTS, LOW, MID };

// The low pivot's bound (the slot merge's too): what both forms need, flags,
// symmetric adjacency with its slot map, temporaries of the bins and the
// aggregation.
static int64_t common_bytes(const tc_graph *g) {
    // support per oriented slot and per edge, tri, num, tc, triG
    return 8 * g->m + 24 * (int64_t)(g->n > 0 ? g->n : 1) + 8 * ((int64_t)g->num_graphs + 1);
}
// The caching allocator rounds each block up: by under 512 bytes below 1 MiB, by
// under 2 MiB above; at most 64 blocks, each above 1 MiB taking at least 1 MiB of b.
static int64_t with_rounding(int64_t b) {
    const int64_t big = (b >> 20) < 64 ? (b >> 20) : 64;
    return b + 64 * 512 + big * ((int64_t)2 << 20);
}
static int64_t low_bytes(const tc_graph *g) {
    return with_rounding(common_bytes(g) + 34 * g->m + 40 * (int64_t)(g->n > 0 ? g->n : 1));
}

// Where rows are short enough for the slot merge: whether its hits, an atomic add
// to a row of another workgroup each, cost more than the middle pivot.  Device time
// in ns per edge, merge and middle pivot, by triangles per edge: 0.6 0.06 / 0.30;
// 5.8 0.35 / 0.37; 7.2 0.30 / 0.36; 10 (R-MAT scale 12, 256 times) 0.45 / 0.31; 19
// (K_60) 0.83 / 0.31; 33 (K_100) 1.34 / 0.45; that is about 0.06 + 0.038 t against
// 0.34, and the middle pivot's launches take 70 us more.
static bool merge_hits_dear(const tc_graph *g) {
    return (double)g->m * (0.038 * g->tri_per_edge - 0.28) > 70e3;
}

// The form that AUTO (or the tuning) takes for this graph.
static Form choose_form(const tc_graph *g, const tc_tuning &t) {
    if (t.algorithm != TC_ALGO_AUTO)
        return t.algorithm == TC_ALGO_MID_PIVOT ? Form::MID : Form::LOW;
    // the slot merge (tc_slots.hip, a low-pivot form without tables) where every
    // oriented row is short
    const bool short_rows = g->max_dplus <= TC_SLOTS_MAX_DPLUS;
    const Form few = short_rows ? Form::SLOTS : Form::LOW;
    if (g->m < AUTO_MID_MIN_EDGES || (short_rows && !merge_hits_dear(g))) return few;
    if (tc_low_bytes_promised(g) && tc_mid_most_bytes(g) > low_bytes(g)) return few;
    return Form::MID;
}

tc_status tc_count_bytes(tc_graph *g, const tc_tuning *tin, hipStream_t s, int64_t *bytes) {
    tc_tuning t;
    if (tin) t = *tin; else tc_tuning_default(&t);
    if (!tuning_valid(&t)) return TC_ERR_INVALID_ARG;
    const int64_t m = g->m, nn = g->n > 0 ? g->n : 1;
    const bool promised = t.algorithm == TC_ALGO_AUTO && tc_low_bytes_promised(g);
    if (m == 0 || g->max_dplus < 2 || promised || choose_form(g, t) != Form::MID) {
        *bytes = low_bytes(g);
        return TC_OK;
    }
    int64_t words = 0;
    TC_TRY(tc_mid_bit_words(g, &words, s));
    // transposition (pair lists and offsets), bit matrices with their row
    // records and offsets, the 16-bit columns; temporaries of the
    // transposition sort, work-item lists, support reordering and
    // aggregation, all counted at once
    *bytes = with_rounding(common_bytes(g) + 8 * m + 8 * (nn + 1) + 4 * (words + 4) + 16 * nn +
                           8 * (nn + 1) + 2 * (m + 66) + 30 * m + 96 * nn);
    return TC_OK;
}

tc_status tc_count(tc_graph *g, const tc_tuning *tin, hipStream_t s) {
    tc_tuning t;
    if (tin) t = *tin; else tc_tuning_default(&t);
    if (!tuning_valid(&t)) return TC_ERR_INVALID_ARG;
    const int64_t m = g->m;
    g->slots_used = false;
    if (!g->osup) TC_TRY(tc_graph_alloc(g, &g->osup, m, s));
    if (!g->triG) TC_TRY(tc_graph_alloc(g, &g->triG, g->num_graphs + 1, s));
    // triG[num_graphs] is the scratch total of triangles found by the count
    unsigned long long *found = (unsigned long long *)(g->triG + g->num_graphs);
    Form form = choose_form(g, t);
    if (g->single && m > 0 && form == Form::SLOTS) {  // one launch, aggregation included
        g->algo_used = TC_ALGO_LOW_PIVOT;
        g->slots_used = true;
        g->light_max = t.light_max_dplus;
        g->huge_min = 0x7FFFFFFF;
        tc_prof_mark(g, 5, s);
        TC_TRY(tc_single_count(g, s));
        for (int k = 6; k <= 9; ++k) tc_prof_mark(g, k, s);
        return TC_OK;
    }
    TC_TRY(tc_zero({{g->osup, m > 0 ? m : 1}, {found, 2}}, s));
    if (m == 0 || g->max_dplus < 2) {
        g->light_max = t.light_max_dplus;
        g->huge_min = 0x7FFFFFFF;
        for (int k = 5; k <= 9; ++k) tc_prof_mark(g, k, s);
        for (int k = 12; k <= 14; ++k) tc_prof_mark(g, k, s);
        return TC_OK;
    }

    // The heavy kernel's table and counters must fit one workgroup's LDS:
    // clamp the table size to what this device allows.
    int dev = 0, lds_limit = 65536;
    TC_HIP(hipGetDevice(&dev));
    TC_HIP(hipDeviceGetAttribute(&lds_limit, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    int max_entries = t.lds_max_entries;
    while (max_entries > 1024 && heavy_bytes(max_entries / 2) > (size_t)lds_limit) max_entries >>= 1;
    // AUTO, above the slot merge: the middle pivot streams fewer candidates
    // (the oriented wedges), but its transposition, work items and fold cost a
    // fixed number of launches and a host round trip.
    g->algo_used = form == Form::MID ? TC_ALGO_MID_PIVOT : TC_ALGO_LOW_PIVOT;
    if (form == Form::MID) {
        const tc_status st = tc_count_mid(g, t, lds_limit, max_entries, found, s);
        if (!tc_no_memory(st) || !tc_mid_may_yield(g, t)) return st;
        // its arrays do not fit: the other forms do without
        tc_mid_release(g, s);
        g->algo_used = TC_ALGO_LOW_PIVOT;
        form = g->max_dplus <= TC_SLOTS_MAX_DPLUS ? Form::SLOTS : Form::LOW;
    }
    if (form == Form::SLOTS) {
        g->slots_used = true;
        g->light_max = t.light_max_dplus;
        g->huge_min = 0x7FFFFFFF;
        tc_prof_mark(g, 5, s);
        TC_TRY(tc_count_slots(g, found, s));
        for (int k = 6; k <= 9; ++k) tc_prof_mark(g, k, s);
        return TC_OK;
    }
    const int light_max = t.light_max_dplus;
    // heavy rows: light_max < d+ < huge_min (table at most half full); the
    // three bins must not overlap, whatever the knobs
    int huge_min = max_entries / 2 + 1;
    if (huge_min <= light_max) huge_min = light_max + 1;
    tc_scratch tmp(s);
    int32_t *rows = nullptr, *heavy = nullptr, *huge = nullptr;
    uint32_t *cnt = nullptr;
    // the longest row says which bins can hold rows at all
    const bool any_heavy = g->max_dplus > light_max, any_huge = g->max_dplus >= huge_min;
    TC_TRY(tmp.get(&rows, g->n));
    TC_TRY(tmp.get(&heavy, any_heavy ? g->n : 1));
    TC_TRY(tmp.get(&huge, any_huge ? g->n : 1));
    TC_TRY(tmp.get(&cnt, 3));
    TC_TRY(tc_zero({{cnt, 3}}, s));
    k_bin_rows<<<(unsigned)tc_div_up(g->n, BR_TILE), BK, 0, s>>>(g->n, g->orp, light_max, huge_min,
                                                                rows, heavy, huge, cnt);
    TC_LAUNCHED();
    g->light_max = light_max;
    g->huge_min = huge_min;
    tc_prof_mark(g, 5, s);

    {
        // tables and counters for the longest light row there is; as many
        // workgroups as stay resident (8 of 4 wavefronts per CU), each taking
        // rows in turn
        const int dcap = g->max_dplus < light_max ? g->max_dplus : light_max;
        const size_t per_wave = light_wave_bytes(dcap);
        int wpb = t.light_block / TC_WAVE;
        while (wpb > 1 && (size_t)wpb * per_wave > (size_t)lds_limit) --wpb;
        const int block = wpb * TC_WAVE;
        const size_t lds = (size_t)wpb * per_wave;
        int64_t blocks = tc_div_up(g->n, wpb);
        if (blocks > 8192 / wpb) blocks = 8192 / wpb;
        k_count_light<<<(unsigned)blocks, block, lds, s>>>(g->orp, g->ocol, rows, cnt, dcap, g->osup,
                                                         found);
        TC_LAUNCHED();
    }
    tc_prof_mark(g, 6, s);
    if (any_heavy) {
        // every heavy row has light_max < d+ < huge_min and d+ <= max d+
        const int hmax = g->max_dplus < huge_min - 1 ? g->max_dplus : huge_min - 1;
        const size_t lds = heavy_bytes(hmax);
        const int64_t blocks = g->n < 8192 ? g->n : 8192;
        k_count_heavy<false><<<(unsigned)blocks, t.heavy_block, lds, s>>>(
            g->orp, g->ocol, heavy, cnt + 1, hmax, g->osup, found);
        TC_LAUNCHED();
    }
    tc_prof_mark(g, 7, s);
    if (any_huge) {
        const int64_t blocks = g->n < 8192 ? g->n : 8192;
        k_count_heavy<true><<<(unsigned)blocks, t.heavy_block, 0, s>>>(g->orp, g->ocol, huge, cnt + 2,
                                                                      0, g->osup, found);
        TC_LAUNCHED();
    }
    tc_prof_mark(g, 8, s);
    tc_prof_mark(g, 9, s);  // the low-pivot form has no fold step
    return TC_OK;
}

// ---------------------------------------------------------------------------
// Work measures of the orientation (instrumentation).
// ---------------------------------------------------------------------------
namespace {

__global__ void k_work_stats(int32_t n, const int64_t *__restrict__ orp,
                             const int32_t *__restrict__ ocol, int light_max, int huge_min,
                             bool low_bins, unsigned long long *__restrict__ acc) {
    // per-thread sums of the 12 words, added once per wavefront: the words
    // are shared by every row
    unsigned long long sums[12] = {};
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n;
         r += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = orp[r], e = orp[r + 1];
        const int64_t d = e - b;
        if (d == 0) continue;
        unsigned long long cand = 0, merge = 0;
        for (int64_t k = b; k < e; ++k) {
            const int32_t u = ocol[k];
            const int64_t du = orp[u + 1] - orp[u];
            cand += du;
            merge += d + du;
        }
        const int bin = d < 2 ? -1 : (d <= light_max ? 0 : (d < huge_min ? 1 : 2));
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (bin == q && low_bins) {
                sums[q] += 1ull;
                sums[3 + q] += cand;
                sums[8 + q] += (unsigned long long)d;
            }
        }
        sums[6] += merge;
        sums[7] += (unsigned long long)(d * (d - 1) / 2);
        sums[11] += cand;
    }
#pragma unroll
    for (int q = 0; q < 12; ++q) {
        const unsigned long long t = tc_wave_sum(sums[q]);
        if (__lane_id() == 0 && t) atomicAdd(&acc[q], t);
    }
}

}  // namespace

tc_status tc_work_stats(tc_graph *g, int64_t *stats, hipStream_t s) {
    for (int i = 0; i < TC_NUM_WORK_STATS; ++i) stats[i] = 0;
    stats[TC_STAT_N] = g->n;
    stats[TC_STAT_M] = g->m;
    stats[TC_STAT_MAX_DPLUS] = g->max_dplus;
    if (g->n == 0 || g->m == 0) return TC_OK;
    tc_scratch tmp(s);
    unsigned long long *acc = nullptr;
    TC_TRY(tmp.get(&acc, 15));
    TC_HIP(hipMemsetAsync(acc, 0, 15 * sizeof(unsigned long long), s));
    int light_max = g->light_max > 0 ? g->light_max : 64;
    int huge_min = g->huge_min > 0 ? g->huge_min : 0x7FFFFFFF;
    const bool mid = g->algo_used != TC_ALGO_LOW_PIVOT;
    const unsigned wg = grid_for(g->n) < 4096u ? grid_for(g->n) : 4096u;
    k_work_stats<<<wg, BK, 0, s>>>(g->n, g->orp, g->ocol, light_max, huge_min, !mid,
                                               acc);
    TC_LAUNCHED();
    if (mid) TC_TRY(tc_mid_stats(g, acc, s));
    unsigned long long h[15];
    uint64_t tri = 0;
    TC_HIP(hipMemcpyAsync(h, acc, sizeof(h), hipMemcpyDeviceToHost, s));
    if (g->triG) TC_HIP(hipMemcpyAsync(&tri, g->triG + g->num_graphs, 8, hipMemcpyDeviceToHost, s));
    TC_HIP(hipStreamSynchronize(s));
    stats[TC_STAT_ROWS_LIGHT] = (int64_t)h[0];
    stats[TC_STAT_ROWS_HEAVY] = (int64_t)h[1];
    stats[TC_STAT_ROWS_HUGE] = (int64_t)h[2];
    stats[TC_STAT_CAND_LIGHT] = (int64_t)h[3];
    stats[TC_STAT_CAND_HEAVY] = (int64_t)h[4];
    stats[TC_STAT_CAND_HUGE] = (int64_t)h[5];
    stats[TC_STAT_MERGE_WORK] = (int64_t)h[6];
    stats[TC_STAT_WEDGES] = (int64_t)h[7];
    stats[TC_STAT_TRIANGLES] = (int64_t)tri;
    stats[TC_STAT_EDGES_LIGHT] = (int64_t)h[8];
    stats[TC_STAT_EDGES_HEAVY] = (int64_t)h[9];
    stats[TC_STAT_EDGES_HUGE] = (int64_t)h[10];
    stats[TC_STAT_W_HASH] = (int64_t)h[11];
    stats[TC_STAT_ALGORITHM] = mid ? TC_ALGO_MID_PIVOT : TC_ALGO_LOW_PIVOT;
    stats[TC_STAT_CAND_HEAVY_16] = (int64_t)h[12];
    stats[TC_STAT_EDGES_HEAVY_16] = (int64_t)h[13];
    stats[TC_STAT_ROWS_HEAVY_16] = (int64_t)h[14];
    return TC_OK;
}
