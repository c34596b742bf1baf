// Graph build on the device: normalisation into the canonical edge list
// and the symmetric CSR, the degree ordering, and the degree-ordered
// orientation.
//
//  1. Pack every pair as the 64-bit key (min << bits) | max (self-loops
//     become a sentinel above every real key), radix sort, keep first
//     occurrences: canonical edges (u < v) in lexicographic order.
//  2. Symmetric CSR in original ids.  Row x is [smaller neighbours] then
//     [larger neighbours]; the larger ones are the run of canonical edges
//     with eu = x (already sorted), the smaller ones come from a stable
//     sort of (ev, e) -- the transpose -- which lists them by increasing eu.
//  3. Degree ordering π (Sec. "Notation"): position in the order by
//     (degree, id), from a stable sort of degrees over ids in id order.
//  4. Orientation: each canonical edge becomes (π(low), π(high)); a sort of
//     these packed keys yields the oriented CSR whose row r lists the
//     higher-ordered neighbours N_H of the rank-r vertex, ascending.  This
//     is the paper's split of N(v) into N_L(v) | N_H(v) (Lemma 1's proof),
//     stored as its own compact array for the counting kernels.
#include <stdlib.h>

#include "tc_internal.h"

namespace {

constexpr int BK = 256;

static inline unsigned grid_for(int64_t n, int block = BK) {
    int64_t g = tc_div_up(n, block);
    if (g < 1) g = 1;
    if (g > 0x7FFFFFFF) g = 0x7FFFFFFF;
    return (unsigned)g;
}

#define GRID_STRIDE(i, n) \
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

// The last index g in [lo, hi] with off[g] <= x.
__device__ __forceinline__ int32_t last_at_or_below(const int64_t *__restrict__ off, int32_t lo,
                                                    int32_t hi, int64_t x) {
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (off[mid] <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The graphs of a workgroup's first and last element (x0 <= x1), found once, so
// that its elements search between them: a step or none, where each had searched
// all graphs (1.8e7 pairs of 512 graphs: 126 us, 57 so with 8 pairs per thread).  Every thread calls.
__device__ __forceinline__ void graph_range(const int64_t *__restrict__ off, int32_t G, int64_t x0,
                                            int64_t x1, int32_t (&lds)[2], int32_t &lo, int32_t &hi) {
    if (threadIdx.x == 0) lds[0] = last_at_or_below(off, 0, G - 1, x0);
    if (threadIdx.x == TC_WAVE) lds[1] = last_at_or_below(off, 0, G - 1, x1);
    __syncthreads();
    lo = lds[0];
    hi = lds[1];
}

// Pair -> packed canonical key (lower id << vbits | higher id).  For a batch, pair
// i belongs to the graph g with pair_off[g] <= i < pair_off[g+1]; its ids are
// local; the lower one gets the graph's first global vertex id added and the
// higher one stays local, whose vbits are fewer.
constexpr int64_t KEYS_MANY = (int64_t)1 << 20;  // from here on 8 pairs per thread

template <int ITEMS>
__global__ __launch_bounds__(BK) void k_make_keys(const int32_t *__restrict__ src,
                                                  const int32_t *__restrict__ dst, int64_t P,
                                                  int32_t n, int vbits, uint64_t sentinel,
                                                  const int64_t *__restrict__ pair_off,
                                                  const int64_t *__restrict__ vtx_off, int32_t G,
                                                  uint64_t *__restrict__ keys,
                                                  uint32_t *__restrict__ err) {
    __shared__ int32_t range[2];
    const int64_t i0 = (int64_t)blockIdx.x * (BK * ITEMS);
    int32_t x[ITEMS], y[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = i0 + it * BK + threadIdx.x;
        x[it] = i < P ? src[i] : 0;
        y[it] = i < P ? dst[i] : 0;
    }
    int32_t g0 = 0, g1 = 0;
    if (pair_off != nullptr)
        graph_range(pair_off, G, i0, i0 + BK * ITEMS < P ? i0 + BK * ITEMS - 1 : P - 1, range, g0, g1);
    bool bad = false;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = i0 + it * BK + threadIdx.x;
        if (i >= P) break;
        int64_t lim = n, base = 0;
        if (pair_off != nullptr) {
            const int32_t g = last_at_or_below(pair_off, g0, g1, i);
            base = vtx_off[g];
            lim = vtx_off[g + 1] - base;
        }
        const int64_t a = x[it], b = y[it];
        uint64_t key = sentinel;
        if (a < 0 || a >= lim || b < 0 || b >= lim) bad = true;
        else if (a != b)
            key = (uint64_t)((a < b ? a : b) + base) << vbits | (uint64_t)(a < b ? b : a);
        keys[i] = key;
    }
    if (bad) atomicOr(err, 1u);
}

// Deduplication as a two-pass compaction over tiles of UQ_TILE sorted keys:
// k_unique_count counts each tile's canonical edges (the first key of every
// run of equal keys, sentinels excluded), the tile counts are scanned, and
// k_unique_emit recomputes the flags, places them by a workgroup scan and
// stores the tile's edges side by side.  Every key is read twice and every
// edge written once; no per-key flag or position array goes to memory.
constexpr int UQ_BLOCK = 256;
constexpr int UQ_ITEMS = 16;
constexpr int UQ_TILE = UQ_BLOCK * UQ_ITEMS;

__device__ __forceinline__ bool first_of_run(const uint64_t *__restrict__ keys, int64_t i,
                                             uint64_t k, uint64_t sentinel) {
    return k != sentinel && (i == 0 || keys[i - 1] != k);
}

__global__ __launch_bounds__(UQ_BLOCK) void k_unique_count(const uint64_t *__restrict__ keys,
                                                           int64_t P, uint64_t sentinel,
                                                           uint32_t *__restrict__ cnt) {
    __shared__ uint32_t red[UQ_BLOCK / TC_WAVE];
    const int64_t base = (int64_t)blockIdx.x * UQ_TILE;
    uint32_t c = 0;
#pragma unroll
    for (int it = 0; it < UQ_ITEMS; ++it) {
        const int64_t i = base + it * UQ_BLOCK + threadIdx.x;
        if (i < P) c += first_of_run(keys, i, keys[i], sentinel) ? 1u : 0u;
    }
    c = tc_wave_sum(c);
    if (__lane_id() == 0) red[threadIdx.x / TC_WAVE] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int w = 0; w < UQ_BLOCK / TC_WAVE; ++w) t += red[w];
        cnt[blockIdx.x] = t;
    }
}

// Writes the canonical edges of each tile at tile_off[tile] and, in the same
// pass, the run [us[u], ue[u]) of the edges whose smaller end is u (edges
// come sorted by it).  us and ue start zeroed.  m: all edges.
__global__ __launch_bounds__(UQ_BLOCK) void k_unique_emit(const uint64_t *__restrict__ keys,
                                                          int64_t P, uint64_t sentinel, int vbits,
                                                          const int64_t *__restrict__ vtx_off,
                                                          int32_t G,
                                                          const uint32_t *__restrict__ tile_off,
                                                          int64_t m, int32_t *__restrict__ eu,
                                                          int32_t *__restrict__ ev,
                                                          uint32_t *__restrict__ us,
                                                          uint32_t *__restrict__ ue) {
    constexpr int W = UQ_BLOCK / TC_WAVE;
    __shared__ int32_t su[UQ_TILE], sv[UQ_TILE];
    __shared__ uint32_t cnt[UQ_ITEMS * W];  // flags per (item, wavefront), then their prefix
    __shared__ uint32_t total;
    __shared__ int32_t range[2];
    static_assert(UQ_ITEMS * W == TC_WAVE, "a wavefront scans the counts");
    const uint64_t mask = (1ull << vbits) - 1;
    const int64_t base = (int64_t)blockIdx.x * UQ_TILE;
    const int w = threadIdx.x / TC_WAVE;
    const int lane = __lane_id();
    const uint64_t lt = tc_lanemask_lt();
    // element it * UQ_BLOCK + threadIdx.x of the tile: a wavefront holds 64
    // consecutive elements per item, and tile order is (item, wavefront, lane)
    uint64_t k[UQ_ITEMS], prev[UQ_ITEMS], fl[UQ_ITEMS];
#pragma unroll
    for (int it = 0; it < UQ_ITEMS; ++it) {
        const int64_t i = base + it * UQ_BLOCK + threadIdx.x;
        k[it] = i < P ? keys[i] : sentinel;
        prev[it] = (i > 0 && i < P) ? keys[i - 1] : sentinel;
        fl[it] = __ballot(k[it] != sentinel && (i == 0 || prev[it] != k[it]));
        if (lane == 0) cnt[it * W + w] = (uint32_t)__popcll(fl[it]);
    }
    __syncthreads();
    if (w == 0) {
        const uint32_t c = cnt[lane], incl = tc_wave_incl_scan(c);
        cnt[lane] = incl - c;
        if (lane == TC_WAVE - 1) total = incl;
    }
    int32_t g0 = 0, g1 = 0;
    if (vtx_off != nullptr) {
        const int64_t last = base + UQ_TILE < P ? base + UQ_TILE - 1 : P - 1;
        graph_range(vtx_off, G, (int64_t)(keys[base] >> vbits), (int64_t)(keys[last] >> vbits), range,
                    g0, g1);
    }
    __syncthreads();
    const uint32_t p0 = tile_off[blockIdx.x];
#pragma unroll
    for (int it = 0; it < UQ_ITEMS; ++it) {
        if ((fl[it] >> lane) & 1ull) {
            const uint32_t lp = cnt[it * W + w] + (uint32_t)__popcll(fl[it] & lt);
            const uint32_t u = (uint32_t)(k[it] >> vbits);
            int64_t v = (int64_t)(k[it] & mask);
            if (vtx_off != nullptr) v += vtx_off[last_at_or_below(vtx_off, g0, g1, u)];
            su[lp] = (int32_t)u;
            sv[lp] = (int32_t)v;
            // prev is the previous distinct key (sentinels sort last)
            const uint32_t pu = (uint32_t)(prev[it] >> vbits);
            if (base + it * UQ_BLOCK + threadIdx.x == 0) {
                us[u] = 0;
            } else if (pu != u) {
                us[u] = p0 + lp;
                ue[pu] = p0 + lp;
            }
            if (p0 + lp + 1 == m) ue[u] = (uint32_t)m;  // the last run
        }
    }
    __syncthreads();
    const uint32_t tot = total;
    for (uint32_t j = threadIdx.x; j < tot; j += UQ_BLOCK) {
        eu[p0 + j] = su[j];
        ev[p0 + j] = sv[j];
    }
}

// A CSR given as simple and sorted: each row strictly increasing, ids in
// [0, n), no self-loop (checked: a violation sets err).  Its entries above
// the diagonal, row by row, are the canonical edges in order, so the edge
// list is an ordered compaction of the entries, in two passes like the one
// above: CT_COUNT counts each tile's upper entries (and checks them), CT_EMIT
// writes them at the tile's offset with the run [us[v], ue[v]) of every row
// that has some.
//
// What bounds it: one read of col per pass and the edge stores.  A tile is a
// slice of CT_TILE steps of the merge of the row ends with the entries, found
// by a binary search, so every workgroup has the same work whatever the row
// lengths are: a thread per row made the hubs a serial chain (R-MAT scale 16,
// 1.82 M stored entries: 1846 + 675 us; as tiles 15 + 14 us).
constexpr int CT_BLOCK = 256;
constexpr int CT_ITEMS = 16;
constexpr int CT_TILE = CT_BLOCK * CT_ITEMS;

// Rows consumed after `diag` steps of the merge (ties: the row end first).
__device__ __forceinline__ int64_t csr_split(const int64_t *__restrict__ rp, int64_t n, int64_t nnz,
                                             int64_t diag) {
    int64_t lo = diag > nnz ? diag - nnz : 0, hi = diag < n ? diag : n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (rp[mid + 1] <= diag - mid - 1) lo = mid + 1; else hi = mid;
    }
    return lo;
}

template <bool EMIT>
__global__ __launch_bounds__(CT_BLOCK) void k_csr_upper(
    const int64_t *__restrict__ rp, const int32_t *__restrict__ col, int32_t n, int64_t nnz,
    uint32_t *__restrict__ cnt, const uint32_t *__restrict__ tile_off, int32_t *__restrict__ eu,
    int32_t *__restrict__ ev, uint32_t *__restrict__ us, uint32_t *__restrict__ ue,
    uint32_t *__restrict__ err) {
    constexpr int W = CT_BLOCK / TC_WAVE;
    // row of each entry of the tile, one pad word per 16 so that the threads'
    // runs of 16 start in different banks
    __shared__ int32_t row[CT_TILE + CT_TILE / CT_ITEMS];
    __shared__ int64_t split[2];
    __shared__ int32_t wmax[W];
    __shared__ uint32_t wcnt[CT_ITEMS * W];
    const auto px = [](int i) { return i + i / CT_ITEMS; };
    const int tid = threadIdx.x, lane = __lane_id(), w = tid / TC_WAVE;
    const int64_t d0 = (int64_t)blockIdx.x * CT_TILE;
    const int64_t d1 = d0 + CT_TILE < n + nnz ? d0 + CT_TILE : n + nnz;
    if (tid < 2) split[tid] = csr_split(rp, n, nnz, tid == 0 ? d0 : d1);
    for (int i = tid; i < CT_TILE; i += CT_BLOCK) row[px(i)] = -1;
    __syncthreads();
    const int64_t i0 = split[0], i1 = split[1];
    const int64_t j0 = d0 - i0;
    const int ne = (int)(d1 - i1 - j0);  // entries of the tile
    // each non-empty row that starts inside the tile marks its first entry;
    // the entries before the first mark belong to row i0
    for (int64_t r = i0 + 1 + tid; r <= i1 && r < n; r += CT_BLOCK) {
        const int64_t a = rp[r];
        if (a < rp[r + 1] && a - j0 < ne) row[px((int)(a - j0))] = (int32_t)r;
    }
    __syncthreads();
    // inclusive maximum over the entries (rows only grow)
    int32_t v[CT_ITEMS], mx = -1;
#pragma unroll
    for (int k = 0; k < CT_ITEMS; ++k) {
        const int32_t x = row[px(tid * CT_ITEMS + k)];
        mx = x > mx ? x : mx;
        v[k] = mx;
    }
    int32_t incl = mx;
#pragma unroll
    for (int off = 1; off < TC_WAVE; off <<= 1) {
        const int32_t y = __shfl_up(incl, off, TC_WAVE);
        if (lane >= off && y > incl) incl = y;
    }
    if (lane == TC_WAVE - 1) wmax[w] = incl;
    int32_t before = __shfl_up(incl, 1, TC_WAVE);
    if (lane == 0) before = -1;
    __syncthreads();
    before = before > (int32_t)i0 ? before : (int32_t)i0;
    for (int q = 0; q < w; ++q) before = wmax[q] > before ? wmax[q] : before;
#pragma unroll
    for (int k = 0; k < CT_ITEMS; ++k)
        row[px(tid * CT_ITEMS + k)] = v[k] > before ? v[k] : before;
    __syncthreads();
    // entries it * CT_BLOCK + tid: a wavefront takes 64 neighbours per item
    int32_t x[CT_ITEMS], r[CT_ITEMS];
    uint64_t fl[CT_ITEMS];
    uint32_t head = 0;  // bit it: the entry opens its row's run of upper entries
    bool bad = false;
#pragma unroll
    for (int it = 0; it < CT_ITEMS; ++it) {
        const int i = it * CT_BLOCK + tid;
        const bool in = i < ne;
        x[it] = in ? col[j0 + i] : -1;
        r[it] = in ? row[px(i)] : 0;
        // the entry before, if it is in the same row
        int32_t px_ = -1;
        if (in) {
            const bool same = i > 0 ? row[px(i - 1)] == r[it] : j0 > rp[r[it]];
            if (same) px_ = col[j0 + i - 1];
            if constexpr (!EMIT)
                bad |= x[it] < 0 || x[it] >= n || x[it] == r[it] || (same && px_ >= x[it]);
        }
        fl[it] = __ballot(in && x[it] > r[it]);
        head |= (px_ <= r[it] ? 1u : 0u) << it;
        if (lane == 0) wcnt[it * W + w] = (uint32_t)__popcll(fl[it]);
    }
    if constexpr (!EMIT) {
        if (bad) atomicOr(err, 1u);
        __syncthreads();
        if (tid < TC_WAVE) {
            static_assert(CT_ITEMS * W == TC_WAVE, "one count per lane");
            const uint32_t c = tc_wave_sum(wcnt[tid]);
            if (tid == 0) cnt[blockIdx.x] = c;
        }
    } else {
        __syncthreads();
        if (tid < TC_WAVE) {
            const uint32_t c = wcnt[tid];
            wcnt[tid] = tc_wave_incl_scan(c) - c;
        }
        __syncthreads();
        const uint32_t p0 = tile_off[blockIdx.x];
        const uint64_t lt = tc_lanemask_lt();
#pragma unroll
        for (int it = 0; it < CT_ITEMS; ++it) {
            if ((fl[it] >> lane) & 1ull) {
                const int i = it * CT_BLOCK + tid;
                const uint32_t p = p0 + wcnt[it * W + w] + (uint32_t)__popcll(fl[it] & lt);
                eu[p] = r[it];
                ev[p] = x[it];
                if ((head >> it) & 1u) us[r[it]] = p;
                const bool last = i + 1 < ne ? row[px(i + 1)] != r[it] : rp[r[it] + 1] == j0 + i + 1;
                if (last) ue[r[it]] = p + 1;
            }
        }
    }
}

// Run boundaries of a sorted id sequence: start/end of each present id.
// start and end must be zeroed first.
template <typename Get>
__global__ void k_runs(Get get, int64_t len, uint32_t *__restrict__ start,
                       uint32_t *__restrict__ end) {
    GRID_STRIDE(i, len) {
        uint32_t x = get(i);
        if (i == 0 || get(i - 1) != x) start[x] = (uint32_t)i;
        if (i == len - 1 || get(i + 1) != x) end[x] = (uint32_t)(i + 1);
    }
}

struct GetU32 {
    const uint32_t *a;
    __device__ uint32_t operator()(int64_t i) const { return a[i]; }
};
struct GetHigh {
    const uint64_t *a;
    int bits;
    __device__ uint32_t operator()(int64_t i) const { return (uint32_t)(a[i] >> bits); }
};

// With vtx_off (several graphs) a vertex's rank key is its graph, then its
// degree: the order within a graph is the same, and as a graph's ranks are
// consecutive, what is read and added to by rank stays inside a graph's few
// hundred KB, which L2 holds, and the sums of the slot merge stay in LDS (512 BA
// graphs with 17.8 M edges, whole call: 4429 to 3401 us).
__global__ void k_degree(int32_t n, const uint32_t *__restrict__ us, const uint32_t *__restrict__ ue,
                         const uint32_t *__restrict__ ls, const uint32_t *__restrict__ le,
                         const int64_t *__restrict__ vtx_off, int32_t G, int dbits,
                         int64_t *__restrict__ deg64, uint32_t *__restrict__ key,
                         uint32_t *__restrict__ dmax) {
    __shared__ uint32_t lds[BK / TC_WAVE];
    uint32_t mx = 0;
    GRID_STRIDE(x, n) {
        uint32_t d = (ue[x] - us[x]) + (le[x] - ls[x]);
        deg64[x] = d;
        key[x] = vtx_off ? (uint32_t)tc_graph_of(vtx_off, G, x) << dbits | d : d;
        mx = d > mx ? d : mx;
    }
    tc_block_raise<BK>(mx, dmax, lds);
}

// Smaller neighbours: transposed entry j = (ev, e) sorted by ev.
__global__ void k_fill_lower(int64_t m, const uint32_t *__restrict__ tkey,
                             const uint32_t *__restrict__ tval, const uint32_t *__restrict__ lstart,
                             const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ eu,
                             int32_t *__restrict__ col, uint32_t *__restrict__ sym2e) {
    GRID_STRIDE(j, m) {
        uint32_t x = tkey[j], e = tval[j];
        int64_t p = row_ptr[x] + (j - (int64_t)lstart[x]);
        col[p] = eu[e];
        sym2e[p] = e;
    }
}

// Larger neighbours: canonical edge e = (x, v) is the (e - ustart[x])-th.
__global__ void k_fill_upper(int64_t m, const int32_t *__restrict__ eu,
                             const int32_t *__restrict__ ev, const uint32_t *__restrict__ ustart,
                             const uint32_t *__restrict__ lstart, const uint32_t *__restrict__ lend,
                             const int64_t *__restrict__ row_ptr, int32_t *__restrict__ col,
                             uint32_t *__restrict__ sym2e) {
    GRID_STRIDE(e, m) {
        uint32_t x = (uint32_t)eu[e];
        int64_t p = row_ptr[x] + (lend[x] - lstart[x]) + (e - (int64_t)ustart[x]);
        col[p] = ev[e];
        sym2e[p] = (uint32_t)e;
    }
}

__global__ void k_invert(const uint32_t *__restrict__ perm, int32_t n, int32_t *__restrict__ perm_out,
                         int32_t *__restrict__ rank) {
    GRID_STRIDE(r, n) {
        uint32_t v = perm[r];
        perm_out[r] = (int32_t)v;
        rank[v] = (int32_t)r;
    }
}

__global__ void k_orient_keys(int64_t m, const int32_t *__restrict__ eu, const int32_t *__restrict__ ev,
                              const int32_t *__restrict__ rank, int bits, uint64_t *__restrict__ okey,
                              uint32_t *__restrict__ oval) {
    GRID_STRIDE(e, m) {
        uint64_t a = (uint32_t)rank[eu[e]], b = (uint32_t)rank[ev[e]];
        uint64_t lo = a < b ? a : b, hi = a < b ? b : a;
        okey[e] = (lo << bits) | hi;
        oval[e] = (uint32_t)e;
    }
}

__global__ void k_orient_split(int64_t m, const uint64_t *__restrict__ okey, int bits,
                               int32_t *__restrict__ ocol, int32_t *__restrict__ orow) {
    const uint64_t mask = (1ull << bits) - 1;
    GRID_STRIDE(k, m) {
        ocol[k] = (int32_t)(okey[k] & mask);
        orow[k] = (int32_t)(okey[k] >> bits);
    }
}

__global__ void k_run_len64(int32_t n, const uint32_t *__restrict__ s, const uint32_t *__restrict__ e,
                            int64_t *__restrict__ len, uint32_t *__restrict__ maxlen) {
    // one atomic per wavefront: a single word hit by every thread serialises
    uint32_t mx = 0;
    GRID_STRIDE(x, n) {
        uint32_t d = e[x] - s[x];
        len[x] = d;
        mx = d > mx ? d : mx;
    }
    mx = tc_wave_max(mx);
    if (__lane_id() == 0 && mx) atomicMax(maxlen, mx);
}

// ---------------------------------------------------------------------------
// Orientation without a global sort (every row at most SEG_MAX entries):
//   pass A  each canonical edge is written once, into the bucket of its
//           lower-ordered endpoint x: (rank of the other end, edge id) at
//           tmp[row_ptr[x] + slot] (a bucket never outgrows x's symmetric
//           row).  The edges are visited twice, in canonical order (runs of
//           the smaller id u) taking those with x = u, and ordered by the
//           larger id (runs of v) taking those with x = v, so a wavefront's
//           entries for one bucket are neighbours and take their slots with
//           one atomic on x's cursor, and are stored side by side;
//   pass B  d+ = the cursors, scanned into the offsets of the rank rows;
//           each bucket is put in order by rank in LDS and written to
//           ocol/o2e, with the row of every slot in orow.
// ---------------------------------------------------------------------------
constexpr int SEG_MAX = 4096;
constexpr int SEG_WAVE = 64;    // buckets up to this many entries: a group of lanes each
constexpr int SEG_SMALL = 256;  // up to this many: k_orient_small; above: bitonic sorts

// Lanes hold consecutive elements of a sequence sorted by x (x is the same
// for neighbouring lanes of one run); the active ones store their entry in
// x's bucket, each run's active lanes taking consecutive slots with one
// atomic.
__device__ __forceinline__ void place_runs(bool valid, int32_t x, bool active, uint64_t entry,
                                           const int64_t *__restrict__ row_ptr,
                                           uint32_t *__restrict__ cursor,
                                           uint64_t *__restrict__ tbuf) {
    const int lane = __lane_id();
    const int32_t prev = __shfl_up(x, 1, TC_WAVE);
    const bool head = valid && (lane == 0 || prev != x);
    const uint64_t heads = __ballot(head);
    const uint64_t acts = __ballot(valid && active);
    const uint64_t upto = (2ull << lane) - 1;             // lanes 0..lane
    const uint64_t below = (1ull << lane) - 1;            // lanes 0..lane-1
    const uint64_t mine = heads & upto;
    const int hl = mine ? 63 - __clzll((long long)mine) : 0;  // head of this lane's run
    uint32_t base = 0;
    if (head) {
        const uint64_t later = heads & ~upto;
        const uint64_t run = (later ? ((later & (0 - later)) - 1) : ~0ull) & ~below;
        const uint32_t cnt = (uint32_t)__popcll(acts & run);
        if (cnt) base = atomicAdd(&cursor[x], cnt);
    }
    base = __shfl(base, hl, TC_WAVE);
    if (valid && active) {
        const uint64_t before = acts & below & ~((1ull << hl) - 1);  // active lanes in [hl, lane)
        tbuf[row_ptr[x] + base + (uint32_t)__popcll(before)] = entry;
    }
}

// Canonical order: edge e = (u, v), u < v; x = u when u is ordered first.
// Also records the rank of u per edge for the second pass.
__global__ void k_place_by_smaller(int64_t m, const int32_t *__restrict__ eu,
                                   const int32_t *__restrict__ ev, const int32_t *__restrict__ rank,
                                   const int64_t *__restrict__ row_ptr,
                                   uint32_t *__restrict__ cursor, uint64_t *__restrict__ tbuf,
                                   uint32_t *__restrict__ rank_u) {
    const int lane = __lane_id();
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x - lane; e0 < m; e0 += stride) {
        const int64_t e = e0 + lane;
        const bool valid = e < m;
        int32_t u = -1;
        bool active = false;
        uint64_t entry = 0;
        if (valid) {
            u = eu[e];
            const uint32_t a = (uint32_t)rank[u], b = (uint32_t)rank[ev[e]];
            rank_u[e] = a;
            active = a < b;
            entry = ((uint64_t)b << 32) | (uint32_t)e;
        }
        place_runs(valid, u, active, entry, row_ptr, cursor, tbuf);
    }
}

// Edges ordered by the larger id v (key v, value e): x = v when v is
// ordered first.
__global__ void k_place_by_larger(int64_t m, const uint32_t *__restrict__ lt_key,
                                  const uint32_t *__restrict__ lt_val,
                                  const int32_t *__restrict__ rank,
                                  const uint32_t *__restrict__ rank_u,
                                  const int64_t *__restrict__ row_ptr,
                                  uint32_t *__restrict__ cursor, uint64_t *__restrict__ tbuf) {
    const int lane = __lane_id();
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t j0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x - lane; j0 < m; j0 += stride) {
        const int64_t j = j0 + lane;
        const bool valid = j < m;
        int32_t v = -1;
        bool active = false;
        uint64_t entry = 0;
        if (valid) {
            v = (int32_t)lt_key[j];
            const uint32_t e = lt_val[j];
            const uint32_t a = rank_u[e], b = (uint32_t)rank[v];
            active = b < a;
            entry = ((uint64_t)a << 32) | e;
        }
        place_runs(valid, v, active, entry, row_ptr, cursor, tbuf);
    }
}

// Adds the oriented wedges of a workgroup's ranks, from base on, to the word of
// the smallest core that holds them.  The sizes lie at least a workgroup's
// ranks apart, so that it meets two words at most.
template <int PER>
__device__ __forceinline__ void core_wedges(int32_t n, int64_t base, const uint32_t (&d)[PER],
                                            unsigned long long *__restrict__ wedges) {
    static_assert(PER * BK <= 2048, "sizes of cores are 2048 apart");
    if (base + PER * BK <= (int64_t)n - tc_core_ranks(TC_CORE_SIZES - 1)) return;
    int j0 = 0;  // the word of the workgroup's highest ranks
    while (base + PER * BK - 1 < (int64_t)n - tc_core_ranks(j0)) ++j0;
    unsigned long long a = 0, b = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t r = base + k * BK + threadIdx.x;
        const unsigned long long w = (unsigned long long)d[k] * (d[k] - 1ull * (d[k] > 0)) / 2;
        if (r >= (int64_t)n - tc_core_ranks(j0)) a += w; else b += w;
    }
    a = tc_wave_sum(a);
    b = tc_wave_sum(b);
    if (__lane_id() != 0) return;
    if (a) atomicAdd(&wedges[j0], a);
    if (b && j0 + 1 < TC_CORE_SIZES) atomicAdd(&wedges[j0 + 1], b);
}

// d+ by rank row, its maximum (info[0]), and the vertices whose buckets a
// wavefront (more than SEG_SMALL entries) or a workgroup (more than SEG_MID)
// sorts: list_mid and list_big in any order, their counts in info[1] and
// info[2].  Taken in rank order, so that the random accesses are 4-byte reads
// and not 8-byte stores; a workgroup takes DL_TILE vertices and at most one
// atomic per word (one per wavefront on info[0] took 180 us from a million
// vertices on, and the lists ten more launches; 17 us so at 2^20).
constexpr int SEG_MID = 1024;  // k_orient_mid's longest bucket
constexpr int DL_TILE = 2048;

// How many triangles an edge has, from TC_SAMPLES edges: each takes two entries of
// its bucket at random and looks for the one of higher rank in the other's bucket.
// Buckets above the slot merge's rows are left out, as the answer is for graphs that
// have none.  The sample's workgroups come first in the launch of the lists, whose
// time it sets with its chain of some nine reads: 13.7 to 15.1 us at 1.2 M vertices,
// 9.3 to 13.7 at 65 k (a search in the canonical edges instead: 16.0, 13.7).
struct SampleArgs {
    unsigned blocks;
    int64_t m;
    const int32_t *eu, *ev, *rank, *perm;
    const int64_t *row_ptr;
    const uint64_t *tbuf;
    unsigned long long *sum;  // twice the triangles that a sampled edge sees, summed
};

__device__ void sample_triangles(const SampleArgs &a, const uint32_t *__restrict__ cursor) {
    constexpr uint32_t U = 8;  // entries looked at together
    const uint32_t s = blockIdx.x * BK + threadIdx.x;
    const int64_t e = a.m * s / TC_SAMPLES;
    const int32_t u = a.eu[e], v = a.ev[e];
    const int32_t x = a.rank[u] < a.rank[v] ? u : v;
    const uint32_t d = cursor[x];
    const uint64_t *const row = a.tbuf + a.row_ptr[x];
    unsigned long long got = 0;
    if (d >= 2 && d <= TC_SLOTS_MAX_DPLUS) {
        const uint32_t h = s * 2654435761u;
        const uint32_t t = (uint32_t)((uint64_t)h * d >> 32);
        uint32_t t2 = t + 1 + (uint32_t)((uint64_t)(h * 2246822519u) * (d - 1) >> 32);
        t2 = t2 < d ? t2 : t2 - d;
        const uint32_t w = (uint32_t)(row[t] >> 32), z = (uint32_t)(row[t2] >> 32);
        const uint32_t hi = w < z ? z : w;
        const int32_t y = a.perm[w < z ? w : z];
        const uint32_t dy = cursor[y];
        const uint64_t *const other = a.tbuf + a.row_ptr[y];
        bool closed = false;
        for (uint32_t k = 0; k < dy && dy <= TC_SLOTS_MAX_DPLUS && !closed; k += U) {
            uint32_t q[U];
#pragma unroll
            for (uint32_t i = 0; i < U; ++i) q[i] = (uint32_t)(other[k + i < dy ? k + i : k] >> 32);
#pragma unroll
            for (uint32_t i = 0; i < U; ++i) closed |= q[i] == hi;
        }
        if (closed) got = d - 1;
    }
    got = tc_wave_sum(got);
    if (__lane_id() == 0 && got) atomicAdd(a.sum, got);
}

__global__ __launch_bounds__(BK) void k_dplus_lists(int32_t n, const uint32_t *__restrict__ cursor,
                                                    const int32_t *__restrict__ perm,
                                                    int64_t *__restrict__ dplus,
                                                    int32_t *__restrict__ list_mid,
                                                    int32_t *__restrict__ list_big,
                                                    uint32_t *__restrict__ info,
                                                    unsigned long long *__restrict__ wedges,
                                                    SampleArgs sample) {
    constexpr int PER = DL_TILE / BK;
    __shared__ uint32_t lds[BK / TC_WAVE + 1];
    if (blockIdx.x < sample.blocks) {
        sample_triangles(sample, cursor);
        return;
    }
    const int64_t base = (int64_t)(blockIdx.x - sample.blocks) * DL_TILE;
    uint32_t d[PER], mx = 0, nmid = 0, nbig = 0;
    int32_t x[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int64_t r = base + k * BK + threadIdx.x;
        x[k] = r < n ? perm[r] : -1;
        d[k] = r < n ? cursor[x[k]] : 0u;
        if (r < n) dplus[r] = d[k];
        mx = d[k] > mx ? d[k] : mx;
        nmid += d[k] > SEG_SMALL && d[k] <= SEG_MID ? 1u : 0u;
        nbig += d[k] > SEG_MID ? 1u : 0u;
    }
    tc_block_raise<BK>(mx, &info[0], lds);
    core_wedges<PER>(n, base, d, wedges);
    if (!__syncthreads_or(nmid | nbig)) return;
    uint32_t pm = tc_block_reserve<BK>(nmid, &info[1], lds);
    uint32_t pb = tc_block_reserve<BK>(nbig, &info[2], lds);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (d[k] > SEG_MID) list_big[pb++] = x[k];
        else if (d[k] > SEG_SMALL) list_mid[pm++] = x[k];
    }
}

// Buckets of 1..SEG_SMALL entries.  A wavefront reads the sizes of up to 64
// consecutive vertices and sorts their buckets by size class (lo, GL],
// GL = 8, 16, 32, 64: GL lanes per bucket, 64 / GL buckets at a time, taken
// from the class's list of lanes in LDS (classes (64, 128] and (128, 256]: the
// whole wavefront, orient_class_wide).  Each lane places its entry by the number
// of smaller keys in its group (keys of a bucket are distinct ranks; groups are
// filled up with the largest value, so that they are read four at a time).  The
// next bucket's entries are loaded while one is sorted.
//
// Bound by the scattered rows (a few lines each) and, where there are few
// wavefronts, by the chain of one bucket after the other: below 2^19 vertices a
// wavefront takes 16, not 64 (R-MAT scale 16: 104 us before, 32; at scale 20, 16
// take 202 us and 64 178, where it was 300; scale 24 2546 to 1882).
struct OrientOut {
    int32_t *ocol;
    uint32_t *o2e;
    int32_t *orow;
};

// The lanes whose bucket is of the class, in order, in lst; their number.
__device__ __forceinline__ int orient_list(bool in, uint8_t *lst) {
    const uint64_t mask = __ballot(in);
    if (in) lst[__popcll(mask & tc_lanemask_lt())] = (uint8_t)__lane_id();
    __builtin_amdgcn_wave_barrier();
    return __popcll(mask);
}

template <int GL>
__device__ __forceinline__ void orient_class(uint32_t dl, uint32_t lo, uint32_t *wsk, uint8_t *lst,
                                             int64_t bl, int32_t rl, int64_t ol,
                                             const uint64_t *__restrict__ tbuf, OrientOut out) {
    static_assert(GL <= SEG_WAVE && TC_WAVE % GL == 0 && GL % 4 == 0, "group size");
    constexpr int GPW = TC_WAVE / GL;
    const int cnt = orient_list(dl > lo && dl <= (uint32_t)GL, lst);
    const int lane = __lane_id();
    const int grp = lane / GL, sl = lane % GL;
    uint32_t *gsk = wsk + grp * GL;
    // this group's it-th vertex, its size (0: none) and this lane's entry
    int j = 0, d = 0;
    uint64_t w = 0;
    const auto load = [&](int at) {
        j = at < cnt ? lst[at] : 0;
        const int64_t bx = __shfl(bl, j, TC_WAVE);
        const int dj = (int)__shfl(dl, j, TC_WAVE);
        d = at < cnt ? dj : 0;
        if (sl < d) w = tbuf[bx + sl];
    };
    load(grp);
    for (int it = 0; it < cnt; it += GPW) {
        const int dc = d;
        const uint64_t wc = w;
        const int32_t rx = __shfl(rl, j, TC_WAVE);
        const int64_t ob = __shfl(ol, j, TC_WAVE);
        load(it + GPW + grp);
        const bool mine = sl < dc;
        const uint32_t key = mine ? (uint32_t)(wc >> 32) : 0xFFFFFFFFu;
        gsk[sl] = key;
        __builtin_amdgcn_wave_barrier();
        if (mine) {
            int pos = 0;
            for (int t = 0; t < dc; t += 4) {
                const uint4 q = *reinterpret_cast<const uint4 *>(gsk + t);
                pos += (q.x < key ? 1 : 0) + (q.y < key ? 1 : 0) + (q.z < key ? 1 : 0) +
                       (q.w < key ? 1 : 0);
            }
            const int64_t k = ob + pos;
            out.ocol[k] = (int32_t)key;
            out.o2e[k] = (uint32_t)wc;
            out.orow[k] = rx;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Buckets of lo < d <= 64 E entries: the whole wavefront, E entries per
// lane, each placed by counting the smaller keys (the keys are read back from
// LDS, the same words for every lane).
template <int E>
__device__ __forceinline__ void orient_class_wide(uint32_t dl, uint32_t lo, uint32_t *wsk,
                                                  uint8_t *lst, int64_t bl, int32_t rl, int64_t ol,
                                                  const uint64_t *__restrict__ tbuf, OrientOut out) {
    const int cnt = orient_list(dl > lo && dl <= (uint32_t)(TC_WAVE * E), lst);
    const int lane = __lane_id();
    int j = 0, d = 0;
    uint64_t w[E] = {};
    const auto load = [&](int at) {
        if (at >= cnt) return;
        j = lst[at];
        d = (int)__shfl(dl, j, TC_WAVE);
        const int64_t b = __shfl(bl, j, TC_WAVE);
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (lane + TC_WAVE * e < d) w[e] = tbuf[b + lane + TC_WAVE * e];
    };
    load(0);
    for (int it = 0; it < cnt; ++it) {
        const int dc = d;
        const int32_t rx = __shfl(rl, j, TC_WAVE);
        const int64_t ob = __shfl(ol, j, TC_WAVE);
        uint32_t key[E], val[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = lane + TC_WAVE * e;
            key[e] = i < dc ? (uint32_t)(w[e] >> 32) : 0xFFFFFFFFu;
            val[e] = (uint32_t)w[e];
            wsk[i] = key[e];
        }
        load(it + 1);
        __builtin_amdgcn_wave_barrier();
        int pos[E];
#pragma unroll
        for (int e = 0; e < E; ++e) pos[e] = 0;
        for (int t = 0; t < dc; t += 4) {
            const uint4 q = *reinterpret_cast<const uint4 *>(wsk + t);
#pragma unroll
            for (int e = 0; e < E; ++e)
                pos[e] += (q.x < key[e] ? 1 : 0) + (q.y < key[e] ? 1 : 0) +
                          (q.z < key[e] ? 1 : 0) + (q.w < key[e] ? 1 : 0);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (lane + TC_WAVE * e < dc) {
                out.ocol[ob + pos[e]] = (int32_t)key[e];
                out.o2e[ob + pos[e]] = val[e];
                out.orow[ob + pos[e]] = rx;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// per: vertices of a wavefront at a time, at most 64
__global__ __launch_bounds__(256) void k_orient_small(
    int32_t n, int per, const int64_t *__restrict__ row_ptr, const uint32_t *__restrict__ cursor,
    const int32_t *__restrict__ rank, const int64_t *__restrict__ orp,
    const uint64_t *__restrict__ tbuf, int32_t *__restrict__ ocol, uint32_t *__restrict__ o2e,
    int32_t *__restrict__ orow) {
    __shared__ uint4 sk[4][SEG_SMALL / 4];
    __shared__ uint8_t lists[4][TC_WAVE];
    const int wv = threadIdx.x / TC_WAVE;
    const int lane = __lane_id();
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    uint32_t *wsk = reinterpret_cast<uint32_t *>(sk[wv]);
    uint8_t *lst = lists[wv];
    const OrientOut out{ocol, o2e, orow};
    for (int64_t x0 = ((int64_t)blockIdx.x * 4 + wv) * per; x0 < n; x0 += nwaves * per) {
        const int64_t xl = x0 + lane;
        const uint32_t dl = lane < per && xl < n ? cursor[xl] : 0u;
        // each lane's vertex: bucket start, rank, oriented row start (the
        // rows of every class in this chunk read them from here)
        int64_t bl = 0, ol = 0;
        int32_t rl = 0;
        if (dl > 0) {
            bl = row_ptr[xl];
            rl = rank[xl];
            ol = orp[rl];
        }
        orient_class<8>(dl, 0, wsk, lst, bl, rl, ol, tbuf, out);
        orient_class<16>(dl, 8, wsk, lst, bl, rl, ol, tbuf, out);
        orient_class<32>(dl, 16, wsk, lst, bl, rl, ol, tbuf, out);
        orient_class<64>(dl, 32, wsk, lst, bl, rl, ol, tbuf, out);
        orient_class_wide<2>(dl, 64, wsk, lst, bl, rl, ol, tbuf, out);
        orient_class_wide<4>(dl, 128, wsk, lst, bl, rl, ol, tbuf, out);
    }
}

// One workgroup per listed vertex (more than SEG_MID entries): the bucket
// as packed (rank << 32 | edge) words, padded with all-ones words to a power
// of two, is put in order by a bitonic sort in LDS.
__global__ __launch_bounds__(256) void k_orient_block(
    const int32_t *__restrict__ list, int64_t nlist, const int64_t *__restrict__ row_ptr,
    const uint32_t *__restrict__ cursor, const int32_t *__restrict__ rank,
    const int64_t *__restrict__ orp, const uint64_t *__restrict__ tbuf,
    int32_t *__restrict__ ocol, uint32_t *__restrict__ o2e, int32_t *__restrict__ orow) {
    __shared__ uint64_t sk[SEG_MAX];
    const int tid = threadIdx.x;
    for (int64_t i = blockIdx.x; i < nlist; i += gridDim.x) {
        const int32_t x = list[i];
        const int32_t rx = rank[x];
        const int64_t ob = orp[rx];
        const int d = (int)cursor[x];
        const int64_t b = row_ptr[x];
        int P = 1;
        while (P < d) P <<= 1;
        for (int j = tid; j < P; j += 256)
            sk[j] = j < d ? tbuf[b + j] : ~0ull;
        __syncthreads();
        for (int k = 2; k <= P; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int t = tid; t < (P >> 1); t += 256) {
                    // t-th pair of this round: lower index a, partner a + j
                    const int a = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                    const uint64_t va = sk[a], vb = sk[a + j];
                    const bool up = (a & k) == 0;
                    if ((va > vb) == up) {
                        sk[a] = vb;
                        sk[a + j] = va;
                    }
                }
                __syncthreads();
            }
        }
        for (int t = tid; t < d; t += 256) {
            const uint64_t w = sk[t];
            ocol[ob + t] = (int32_t)(w >> 32);
            o2e[ob + t] = (uint32_t)w;
            orow[ob + t] = rx;
        }
        __syncthreads();
    }
}

// One wavefront per listed vertex with SEG_SMALL < entries <= SEG_MID: a
// bitonic sort over an LDS buffer of the wavefront's own, so its rounds need
// no workgroup barrier (a wavefront's LDS operations stay in order).

// Bitonic compare-exchange of stage (k, J) on a lane's E consecutive
// elements (global index base + i), for partners inside the lane (J < E).
template <int E, int J>
__device__ __forceinline__ void bitonic_in_lane(uint64_t (&r)[E], int base, int k) {
    if constexpr (J < E) {
#pragma unroll
        for (int i = 0; i < E; ++i) {
            if ((i & J) == 0) {
                const bool up = ((base + i) & k) == 0;
                const uint64_t va = r[i], vb = r[i + J];
                const bool sw = (va > vb) == up;
                r[i] = sw ? vb : va;
                r[i + J] = sw ? va : vb;
            }
        }
    }
}

// One bucket of E * 64 slots (its d entries, padded with all-ones words),
// sorted by one wavefront: each lane keeps E consecutive elements in
// registers, the stages whose partners lie E or more apart go through LDS
// (one store and one load per merge size k), the others stay in registers.
// Slot i sits at LDS word i + i / E, so the lanes' runs of E start in
// different banks.
template <int E>
__device__ __forceinline__ void orient_mid_row(uint64_t *sk, int d, int64_t b, int32_t rx,
                                               int64_t ob, const uint64_t *__restrict__ tbuf,
                                               int32_t *__restrict__ ocol,
                                               uint32_t *__restrict__ o2e,
                                               int32_t *__restrict__ orow) {
    constexpr int P = E * TC_WAVE;
    const int lane = __lane_id();
    const int base = E * lane;
    auto px = [](int i) { return i + i / E; };
    for (int j = lane; j < P; j += TC_WAVE) sk[px(j)] = j < d ? tbuf[b + j] : ~0ull;
    __builtin_amdgcn_wave_barrier();
    uint64_t r[E];
#pragma unroll
    for (int i = 0; i < E; ++i) r[i] = sk[px(base) + i];
    for (int k = 2; k <= P; k <<= 1) {
        if (k > E) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < E; ++i) sk[px(base) + i] = r[i];
            __builtin_amdgcn_wave_barrier();
            for (int j = k >> 1; j >= E; j >>= 1) {
                for (int t = lane; t < (P >> 1); t += TC_WAVE) {
                    const int a = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                    const uint64_t va = sk[px(a)], vb = sk[px(a + j)];
                    const bool up = (a & k) == 0;
                    if ((va > vb) == up) {
                        sk[px(a)] = vb;
                        sk[px(a + j)] = va;
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
#pragma unroll
            for (int i = 0; i < E; ++i) r[i] = sk[px(base) + i];
        }
        // partners inside the lane: J from min(k / 2, E / 2) down to 1
        const int jtop = (k >> 1) < E ? (k >> 1) : (E >> 1);
        if (jtop >= 8) bitonic_in_lane<E, 8>(r, base, k);
        if (jtop >= 4) bitonic_in_lane<E, 4>(r, base, k);
        if (jtop >= 2) bitonic_in_lane<E, 2>(r, base, k);
        bitonic_in_lane<E, 1>(r, base, k);
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < E; ++i) sk[px(base) + i] = r[i];
    __builtin_amdgcn_wave_barrier();
    for (int t = lane; t < d; t += TC_WAVE) {
        const uint64_t w = sk[px(t)];
        ocol[ob + t] = (int32_t)(w >> 32);
        o2e[ob + t] = (uint32_t)w;
        orow[ob + t] = rx;
    }
    __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(256) void k_orient_mid(
    const int32_t *__restrict__ list, int64_t nlist, const int64_t *__restrict__ row_ptr,
    const uint32_t *__restrict__ cursor, const int32_t *__restrict__ rank,
    const int64_t *__restrict__ orp, const uint64_t *__restrict__ tbuf,
    int32_t *__restrict__ ocol, uint32_t *__restrict__ o2e, int32_t *__restrict__ orow) {
    static_assert(SEG_SMALL == 256 && SEG_MID == 1024, "rows of 257..1024 entries: 512 or 1024 slots");
    __shared__ uint64_t sk_all[4][SEG_MID + SEG_MID / 8];
    const int wv = threadIdx.x / TC_WAVE;
    uint64_t *sk = sk_all[wv];
    const int64_t waves = (int64_t)gridDim.x * 4;
    for (int64_t i = (int64_t)blockIdx.x * 4 + wv; i < nlist; i += waves) {
        const int32_t x = list[i];
        const int32_t rx = rank[x];
        const int64_t ob = orp[rx];
        const int d = (int)cursor[x];
        const int64_t b = row_ptr[x];
        if (d <= SEG_MID / 2)
            orient_mid_row<SEG_MID / 2 / TC_WAVE>(sk, d, b, rx, ob, tbuf, ocol, o2e, orow);
        else
            orient_mid_row<SEG_MID / TC_WAVE>(sk, d, b, rx, ob, tbuf, ocol, o2e, orow);
    }
}

}  // namespace

static tc_status orient_sorted(tc_graph *g, hipStream_t s);

void tc_release_transposition(tc_graph *g, hipStream_t s) {
    if (!g->lt_key) return;
    tc_dev_free(g->lt_key, s);
    tc_dev_free(g->lt_val, s);
    g->lt_key = nullptr;
    g->lt_val = nullptr;
    g->bytes -= 2 * sizeof(uint32_t) * (size_t)g->m;
}

tc_status tc_orient(tc_graph *g, hipStream_t s) {
    const int32_t n = g->n;
    const int64_t m = g->m;
    int64_t nn = n > 0 ? n : 1;
    TC_TRY(tc_graph_alloc(g, &g->orp, nn + 1, s));
    // TC_OCOL_PAD trailing entries let the counting kernels load whole
    // 32-entry runs without bounds tests (entries past a run are masked)
    TC_TRY(tc_graph_alloc(g, &g->ocol, m + TC_OCOL_PAD, s));
    TC_TRY(tc_graph_alloc(g, &g->o2e, m, s));
    TC_TRY(tc_graph_alloc(g, &g->orow, m, s));
    g->max_dplus = 0;
    if (m == 0) {
        TC_HIP(hipMemsetAsync(g->orp, 0, sizeof(int64_t) * (nn + 1), s));
        tc_prof_mark(g, 3, s);
        return TC_OK;
    }
    tc_scratch tmp(s);
    int64_t *dplus = nullptr;
    uint32_t *info = nullptr, *cursor = nullptr;
    uint64_t *tbuf = nullptr;
    int32_t *list_mid = nullptr, *list_big = nullptr;
    TC_TRY(tmp.get(&cursor, nn));
    TC_TRY(tmp.get(&tbuf, 2 * m));
    TC_TRY(tmp.get(&dplus, nn));
    // max d+, mid-list count, big-list count; wedges of the cores and the sampled
    // triangles (64-bit)
    constexpr int INFO = 4 + 2 * (TC_CORE_SIZES + 1);
    TC_TRY(tmp.get(&info, INFO));
    TC_TRY(tmp.get(&list_mid, nn));
    TC_TRY(tmp.get(&list_big, nn));
    TC_TRY(tc_zero({{info, INFO}, {cursor, nn}}, s));
    // pass A: buckets of the lower-ordered endpoints
    {
        uint32_t *rank_u = nullptr;
        TC_TRY(tmp.get(&rank_u, m));
        k_place_by_smaller<<<grid_for(m), BK, 0, s>>>(m, g->eu, g->ev, g->rank, g->row_ptr, cursor,
                                                      tbuf, rank_u);
        TC_LAUNCHED();
        k_place_by_larger<<<grid_for(m), BK, 0, s>>>(m, g->lt_key, g->lt_val, g->rank, rank_u,
                                                     g->row_ptr, cursor, tbuf);
        TC_LAUNCHED();
    }
    // with the largest d+ and the lists, whose counts one read-back brings
    unsigned long long *wedges = reinterpret_cast<unsigned long long *>(info + 4);
    const unsigned tiles = (unsigned)tc_div_up(n, DL_TILE);
    const SampleArgs sample{m >= TC_SAMPLE_MIN_EDGES ? TC_SAMPLES / BK : 0u, m, g->eu, g->ev, g->rank,
                            g->perm, g->row_ptr, tbuf, wedges + TC_CORE_SIZES};
    k_dplus_lists<<<tiles + sample.blocks, BK, 0, s>>>(n, cursor, g->perm, dplus, list_mid, list_big, info,
                                                       wedges, sample);
    TC_LAUNCHED();
    uint32_t h_info[4] = {0, 0, 0, 0};
    unsigned long long h_wedges[TC_CORE_SIZES + 1] = {};
    TC_TRY(tc_read({{h_info, info, 3},
                    {&g->max_degree, g->err + 1, 1},
                    {h_wedges, wedges, 2 * (TC_CORE_SIZES + 1)}},
                   s));
    unsigned long long sum = 0;
    for (int j = 0; j < TC_CORE_SIZES; ++j) g->core_wedges[j] = sum += h_wedges[j];
    g->tri_per_edge = (double)h_wedges[TC_CORE_SIZES] / (2.0 * TC_SAMPLES);
    const uint32_t h_max = h_info[0];
    const int64_t nmid = h_info[1], nblk = h_info[2];
    g->max_dplus = (int32_t)h_max;
    // TC_ORIENT_SEG_MAX (environment) lowers the LDS-sort limit, so that the
    // sort-based path can be exercised on small graphs
    uint32_t seg_max = SEG_MAX;
    if (const char *ev = getenv("TC_ORIENT_SEG_MAX")) {
        const long v = strtol(ev, nullptr, 10);
        if (v >= 0 && v < SEG_MAX) seg_max = (uint32_t)v;
    }
    if (h_max > seg_max) {
        TC_TRY(orient_sorted(g, s));
        tc_prof_mark(g, 3, s);
        return TC_OK;
    }
    TC_TRY(tc_scan_i64(dplus, g->orp, n, g->orp + n, s));
    // pass B: each bucket in rank order
    {
        const int per = n < (1 << 19) ? 16 : TC_WAVE;
        const int64_t want = tc_div_up(n, 4 * per);
        const unsigned grid = (unsigned)(want < 65536 ? (want > 0 ? want : 1) : 65536);
        k_orient_small<<<grid, BK, 0, s>>>(n, per, g->row_ptr, cursor, g->rank, g->orp, tbuf, g->ocol,
                                           g->o2e, g->orow);
        TC_LAUNCHED();
    }
    if (nmid > 0) {
        const int64_t blocks = tc_div_up(nmid, 4);
        k_orient_mid<<<(unsigned)(blocks < 1048576 ? blocks : 1048576), BK, 0, s>>>(
            list_mid, nmid, g->row_ptr, cursor, g->rank, g->orp, tbuf, g->ocol, g->o2e, g->orow);
        TC_LAUNCHED();
    }
    if (nblk > 0) {
        k_orient_block<<<(unsigned)(nblk < 1048576 ? nblk : 1048576), BK, 0, s>>>(
            list_big, nblk, g->row_ptr, cursor, g->rank, g->orp, tbuf, g->ocol, g->o2e, g->orow);
        TC_LAUNCHED();
    }
    tc_prof_mark(g, 3, s);
    return TC_OK;
}

// ---------------------------------------------------------------------------
tc_status tc_build_from_pairs(tc_graph *g, const int32_t *d_src, const int32_t *d_dst, int64_t P,
                              const int64_t *d_vtx_off, const int64_t *d_pair_off,
                              int32_t num_graphs, hipStream_t s, const int64_t *simple_rp,
                              const int32_t *simple_col) {
    const int32_t n = g->n;
    const int bits = g->bits;
    // of a batch, the most vertices of a graph: the range of its local ids and
    // degrees
    int64_t most = n;
    if (d_vtx_off) {
        most = 1;
        for (int32_t i = 0; i < num_graphs; ++i) {
            const int64_t c = g->h_vtx_off[i + 1] - g->h_vtx_off[i];
            most = c > most ? c : most;
        }
    }
    // bits of a packed key's higher id (local in a batch: one pass less of the
    // sort for 1.8e7 pairs of 512 graphs)
    const int vbits = d_vtx_off ? tc_bits_for(most > 1 ? (uint64_t)(most - 1) : 1) : bits;
    const uint64_t sentinel = bits + vbits >= 64 ? ~0ull : (1ull << (bits + vbits)) - 1;
    tc_scratch tmp(s);

    TC_TRY(tc_graph_alloc(g, &g->err, 4, s));

    // runs of the edges by smaller end, filled while the canonical edges are
    // written, and by larger end
    int64_t nn = n > 0 ? n : 1;
    uint32_t *ue = nullptr, *ls = nullptr, *le = nullptr;
    TC_TRY(tc_graph_alloc(g, &g->run_us, nn, s));
    uint32_t *us = g->run_us;
    TC_TRY(tmp.get(&ue, nn));
    TC_TRY(tmp.get(&ls, nn));
    TC_TRY(tmp.get(&le, nn));
    TC_TRY(tc_zero({{g->err, 4}, {us, nn}, {ue, nn}, {ls, nn}, {le, nn}}, s));

    // -- 1. canonical edges ---------------------------------------------------
    int64_t m = 0;
    if (simple_rp && n > 0) {
        // a simple sorted CSR of P entries: the upper triangle, no sort and no
        // dedup
        uint32_t *cnt = nullptr, *d_m = nullptr;
        const int64_t tiles = tc_div_up((int64_t)n + P, CT_TILE);
        TC_TRY(tmp.get(&cnt, tiles));
        TC_TRY(tmp.get(&d_m, 1));
        k_csr_upper<false><<<(unsigned)tiles, CT_BLOCK, 0, s>>>(
            simple_rp, simple_col, n, P, cnt, nullptr, nullptr, nullptr, nullptr, nullptr, g->err);
        TC_LAUNCHED();
        TC_TRY(tc_scan_u32(cnt, cnt, tiles, d_m, s));
        uint32_t h_m = 0, h_err = 0;
        TC_TRY(tc_read({{&h_err, g->err, 1}, {&h_m, d_m, 1}}, s));
        if (h_err) return TC_ERR_INVALID_ARG;
        m = h_m;
        TC_TRY(tc_graph_alloc(g, &g->eu, m, s));
        TC_TRY(tc_graph_alloc(g, &g->ev, m, s));
        if (m > 0) {
            k_csr_upper<true><<<(unsigned)tiles, CT_BLOCK, 0, s>>>(
                simple_rp, simple_col, n, P, nullptr, cnt, g->eu, g->ev, us, ue, g->err);
            TC_LAUNCHED();
        }
    } else if (simple_rp) {
        TC_TRY(tc_graph_alloc(g, &g->eu, 0, s));
        TC_TRY(tc_graph_alloc(g, &g->ev, 0, s));
    } else if (P > 0) {
        uint64_t *keys = nullptr, *keys2 = nullptr;
        TC_TRY(tmp.get(&keys, P));
        TC_TRY(tmp.get(&keys2, P));
        // an id out of range makes a sentinel key (dropped like a self
        // loop) and sets err, which is read back with the edge count
        if (P < KEYS_MANY)
            k_make_keys<1><<<grid_for(P), BK, 0, s>>>(d_src, d_dst, P, n, vbits, sentinel, d_pair_off,
                                                      d_vtx_off, num_graphs, keys, g->err);
        else
            k_make_keys<8><<<grid_for(tc_div_up(P, 8)), BK, 0, s>>>(d_src, d_dst, P, n, vbits, sentinel,
                                                                   d_pair_off, d_vtx_off, num_graphs,
                                                                   keys, g->err);
        TC_LAUNCHED();
        TC_TRY(tc_sort_u64(&keys, &keys2, P, bits + vbits, s));
        const int64_t tiles = tc_div_up(P, UQ_TILE);
        uint32_t *tcnt = nullptr, *d_m = nullptr;
        TC_TRY(tmp.get(&tcnt, tiles));
        TC_TRY(tmp.get(&d_m, 1));
        k_unique_count<<<(unsigned)tiles, UQ_BLOCK, 0, s>>>(keys, P, sentinel, tcnt);
        TC_LAUNCHED();
        TC_TRY(tc_scan_u32(tcnt, tcnt, tiles, d_m, s));
        uint32_t h_m = 0, h_err = 0;
        TC_TRY(tc_read({{&h_err, g->err, 1}, {&h_m, d_m, 1}}, s));
        if (h_err) return TC_ERR_VERTEX_RANGE;
        m = h_m;
        TC_TRY(tc_graph_alloc(g, &g->eu, m, s));
        TC_TRY(tc_graph_alloc(g, &g->ev, m, s));
        if (m > 0) {
            k_unique_emit<<<(unsigned)tiles, UQ_BLOCK, 0, s>>>(keys, P, sentinel, vbits, d_vtx_off,
                                                               num_graphs, tcnt, m, g->eu, g->ev, us,
                                                               ue);
            TC_LAUNCHED();
        }
    } else {
        TC_TRY(tc_graph_alloc(g, &g->eu, 0, s));
        TC_TRY(tc_graph_alloc(g, &g->ev, 0, s));
    }
    g->m = m;

    // -- 2. degrees and the symmetric row offsets ------------------------------
    // The adjacency itself (col / sym2e) is filled only when a consumer
    // needs it (tc_ensure_symmetric).
    TC_TRY(tc_graph_alloc(g, &g->row_ptr, (int64_t)n + 1, s));
    // the canonical edges ordered by their larger end (kept for the
    // orientation), whose runs count the edges by larger end
    uint32_t *key = nullptr;
    int64_t *deg64 = nullptr;
    TC_TRY(tmp.get(&key, nn));
    // the rank order's key: (graph, degree) where 32 bits hold both, else the
    // degree, which is below the vertices of its graph
    int dbits = bits;
    bool &by_graph = g->rank_by_graph;
    if (num_graphs > 1 && d_vtx_off) {
        dbits = tc_bits_for((uint64_t)most);
        by_graph = dbits + tc_bits_for((uint64_t)num_graphs) <= 32;
    }
    const int key_bits = by_graph ? dbits + tc_bits_for((uint64_t)num_graphs) : dbits;
    TC_TRY(tmp.get(&deg64, nn));
    if (m > 0) {
        uint32_t *lk2 = nullptr, *lv2 = nullptr;
        TC_TRY(tc_graph_alloc(g, &g->lt_key, m, s));
        TC_TRY(tc_graph_alloc(g, &g->lt_val, m, s));
        TC_TRY(tmp.get(&lk2, m));
        TC_TRY(tmp.get(&lv2, m));
        uint32_t *lk = g->lt_key, *lv = g->lt_val;
        TC_TRY(tc_sort_u32_index((const uint32_t *)g->ev, &lk, &lv, &lk2, &lv2, m, bits, s));
        if (lk != g->lt_key) {  // the result is in the scratch pair: swap ownership
            tmp.exchange(lk, g->lt_key);
            tmp.exchange(lv, g->lt_val);
            g->lt_key = lk;
            g->lt_val = lv;
        }
        k_runs<<<grid_for(m), BK, 0, s>>>(GetU32{g->lt_key}, m, ls, le);
        TC_LAUNCHED();
    }
    if (n > 0) {
        k_degree<<<grid_for(n) < 1024 ? grid_for(n) : 1024, BK, 0, s>>>(
            n, us, ue, ls, le, by_graph ? d_vtx_off : nullptr, num_graphs, dbits, deg64, key, g->err + 1);
        TC_LAUNCHED();
        TC_TRY(tc_scan_i64(deg64, g->row_ptr, n, g->row_ptr + n, s));
    } else {
        TC_HIP(hipMemsetAsync(g->row_ptr, 0, sizeof(int64_t), s));
    }

    tc_prof_mark(g, 1, s);

    // -- 3. degree ordering -------------------------------------------------------
    TC_TRY(tc_graph_alloc(g, &g->rank, nn, s));
    TC_TRY(tc_graph_alloc(g, &g->perm, nn, s));
    if (n > 0) {
        uint32_t *pv = nullptr, *pv2 = nullptr, *dk2 = nullptr;
        TC_TRY(tmp.get(&pv, nn));
        TC_TRY(tmp.get(&pv2, nn));
        TC_TRY(tmp.get(&dk2, nn));
        uint32_t *dk = nullptr;
        TC_TRY(tmp.get(&dk, nn));
        TC_TRY(tc_sort_u32_index(key, &dk, &pv, &dk2, &pv2, n, key_bits, s));
        k_invert<<<grid_for(n), BK, 0, s>>>(pv, n, g->perm, g->rank);
        TC_LAUNCHED();
    }
    tc_prof_mark(g, 2, s);
    return TC_OK;
}

// Orientation by one global sort of the packed (π(low), π(high)) keys; used
// when some row has more than SEG_MAX higher-ordered neighbours.
static tc_status orient_sorted(tc_graph *g, hipStream_t s) {
    const int32_t n = g->n;
    const int64_t m = g->m;
    const int bits = g->bits;
    tc_scratch tmp(s);
    int64_t nn = n > 0 ? n : 1;
    uint64_t *okey = nullptr, *okey2 = nullptr;
    uint32_t *oval2 = nullptr;
    TC_TRY(tmp.get(&okey, m));
    TC_TRY(tmp.get(&okey2, m));
    TC_TRY(tmp.get(&oval2, m));
    uint32_t *oval = g->o2e;
    uint32_t *oval_swap = oval2;
    k_orient_keys<<<grid_for(m), BK, 0, s>>>(m, g->eu, g->ev, g->rank, bits, okey, oval);
    TC_LAUNCHED();
    TC_TRY(tc_sort_u64_u32(&okey, &oval, &okey2, &oval_swap, m, 2 * bits, s));
    if (oval != g->o2e) {
        TC_HIP(hipMemcpyAsync(g->o2e, oval, sizeof(uint32_t) * m, hipMemcpyDeviceToDevice, s));
    }
    k_orient_split<<<grid_for(m), BK, 0, s>>>(m, okey, bits, g->ocol, g->orow);
    TC_LAUNCHED();
    uint32_t *rs = nullptr, *re = nullptr, *d_max = nullptr;
    int64_t *dplus = nullptr;
    TC_TRY(tmp.get(&rs, nn));
    TC_TRY(tmp.get(&re, nn));
    TC_TRY(tmp.get(&dplus, nn));
    TC_TRY(tmp.get(&d_max, 1));
    TC_TRY(tc_zero({{rs, nn}, {re, nn}, {d_max, 1}}, s));
    k_runs<<<grid_for(m), BK, 0, s>>>(GetHigh{okey, bits}, m, rs, re);
    TC_LAUNCHED();
    k_run_len64<<<grid_for(n), BK, 0, s>>>(n, rs, re, dplus, d_max);
    TC_LAUNCHED();
    TC_TRY(tc_scan_i64(dplus, g->orp, n, g->orp + n, s));
    return TC_OK;
}

// ---------------------------------------------------------------------------
tc_status tc_ensure_symmetric(tc_graph *g, hipStream_t s) {
    if (g->col) return TC_OK;
    const int32_t n = g->n;
    const int64_t m = g->m;
    const int64_t nn = n > 0 ? n : 1;
    tc_scratch tmp(s);
    int32_t *col = nullptr;
    uint32_t *sym2e = nullptr;
    TC_TRY(tmp.get(&col, 2 * m));
    TC_TRY(tmp.get(&sym2e, 2 * m));
    const auto take = [&] {
        tc_graph_take(g, &g->col, col, 2 * m, tmp);
        tc_graph_take(g, &g->sym2e, sym2e, 2 * m, tmp);
    };
    if (m == 0) {
        take();
        return TC_OK;
    }
    // the transposition: canonical edges sorted by their larger end (kept
    // from the build unless the middle-pivot count released it), and the
    // run of every vertex in that order
    uint32_t *tkey = g->lt_key, *tval = g->lt_val;
    uint32_t *ls = nullptr, *le = nullptr;
    if (!tkey) {
        uint32_t *tkey2 = nullptr, *tval2 = nullptr;
        TC_TRY(tmp.get(&tkey, m));
        TC_TRY(tmp.get(&tval, m));
        TC_TRY(tmp.get(&tkey2, m));
        TC_TRY(tmp.get(&tval2, m));
        TC_TRY(tc_sort_u32_index((const uint32_t *)g->ev, &tkey, &tval, &tkey2, &tval2, m, g->bits,
                                 s));
    }
    TC_TRY(tmp.get(&ls, nn));
    TC_TRY(tmp.get(&le, nn));
    TC_TRY(tc_zero({{ls, nn}, {le, nn}}, s));
    k_runs<<<grid_for(m), BK, 0, s>>>(GetU32{tkey}, m, ls, le);
    TC_LAUNCHED();
    k_fill_lower<<<grid_for(m), BK, 0, s>>>(m, tkey, tval, ls, g->row_ptr, g->eu, col, sym2e);
    TC_LAUNCHED();
    k_fill_upper<<<grid_for(m), BK, 0, s>>>(m, g->eu, g->ev, g->run_us, ls, le, g->row_ptr, col, sym2e);
    TC_LAUNCHED();
    take();
    tc_release_transposition(g, s);
    return TC_OK;
}
