// Internal declarations of libtc: device helpers, primitive launchers and
// the graph handle.  Not part of the public ABI (include/tc.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tc.h"

#define TC_WAVE 64
#define TC_PROF_MARKS 15
#define TC_OCOL_PAD 64

// ---------------------------------------------------------------------------
// Error plumbing: internal functions return tc_status; HIP failures map to
// TC_ERR_DEVICE (or TC_ERR_OOM for allocation failures).
// ---------------------------------------------------------------------------
#define TC_HIP(call)                                         \
    do {                                                     \
        hipError_t e_ = (call);                              \
        if (e_ != hipSuccess) return tc_map_hip_error(e_);   \
    } while (0)

#define TC_TRY(call)                                         \
    do {                                                     \
        tc_status s_ = (call);                               \
        if (s_ < 0) return s_;                               \
    } while (0)

tc_status tc_map_hip_error(hipError_t e);

// Launch check: kernel launch errors surface through hipGetLastError().
#define TC_LAUNCHED() TC_HIP(hipGetLastError())

__host__ __device__ static inline int64_t tc_div_up(int64_t a, int64_t b) { return (a + b - 1) / b; }

static inline int tc_bits_for(uint64_t max_value) {
    int b = 0;
    while (b < 64 && (max_value >> b) != 0) ++b;
    return b;
}

// ---------------------------------------------------------------------------
// Device memory: the library's caching allocator (tc_api.hip).  A block
// freed on one stream is handed to another stream only after the freeing
// stream's prior work, so temporaries never race with queued kernels.  With
// a limit set (tc_set_memory_limit), an allocation that would push the
// device bytes the library holds past it fails with TC_ERR_BUDGET.
// ---------------------------------------------------------------------------
tc_status tc_dev_alloc(void **p, size_t bytes, hipStream_t s);
// the size of the block that holds bytes
size_t tc_block_size(size_t bytes);
// whether tc_set_memory_limit holds one
bool tc_memory_limited();
// idle: no work that uses the block is pending on any stream
void tc_dev_free(void *p, hipStream_t s, bool idle = false);

// Lives through an entry point: the blocks that the thread frees meanwhile on
// this stream share one event (tc_api.hip).
struct tc_call_scope {
    explicit tc_call_scope(hipStream_t s);
    ~tc_call_scope();
    tc_call_scope(const tc_call_scope &) = delete;
    tc_call_scope &operator=(const tc_call_scope &) = delete;
};

// Reads words (32-bit, at most 64 in all) from device memory to the host and
// waits for the stream.  With step > 0 the words are 64-bit values (two words
// each) that lie step values apart.
constexpr int TC_READ_MAX = 3;
struct tc_read_item {
    void *dst = nullptr;
    const void *src = nullptr;
    int words = 0;
    int64_t step = 0;
};
tc_status tc_read(const tc_read_item (&item)[TC_READ_MAX], hipStream_t s);

template <typename T>
static inline tc_status tc_alloc(T **p, int64_t count, hipStream_t s) {
    size_t bytes = (size_t)(count > 0 ? count : 1) * sizeof(T);
    return tc_dev_alloc((void **)p, bytes, s);
}

// Temporaries of one host function, released (stream-ordered) on exit.
struct tc_scratch {
    static constexpr int MAX = 64;
    hipStream_t s;
    void *ptrs[MAX];
    int n = 0;
    explicit tc_scratch(hipStream_t st) : s(st) {}
    template <typename T>
    tc_status get(T **p, int64_t count) {
        if (n >= MAX) return TC_ERR_INVALID_ARG;
        tc_status r = tc_alloc(p, count, s);
        if (r == TC_OK) ptrs[n++] = (void *)*p;
        return r;
    }
    // p, allocated here, passes to the caller; q (same size) is freed in its place
    void exchange(void *p, void *q) {
        for (int i = 0; i < n; ++i)
            if (ptrs[i] == p) {
                ptrs[i] = q;
                return;
            }
    }
    ~tc_scratch() {
        for (int i = n - 1; i >= 0; --i) tc_dev_free(ptrs[i], s);
    }
};

// ---------------------------------------------------------------------------
// Primitives (tc_scan.hip, tc_sort.hip)
// ---------------------------------------------------------------------------
// Exclusive prefix sum of in[0..n) into out[0..n); if total != nullptr the
// sum of all n inputs is written to *total (device pointer).  in == out is
// allowed.
tc_status tc_scan_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *total,
                      hipStream_t s);
tc_status tc_scan_i64(const int64_t *in, int64_t *out, int64_t n, int64_t *total, hipStream_t s);

// Clears several arrays of 32-bit words with one launch.  A hipMemsetAsync is one
// for whole blocks and one for what is left, so that a call had 13 to 17 of them,
// now 4 (whole calls: 5 M uniform pairs 1198 to 1167 us, a BA graph of 7.5 M edges
// 1234 to 1193).
constexpr int TC_ZERO_MAX = 5;
struct tc_zero_item {
    void *p = nullptr;
    int64_t words = 0;
};
tc_status tc_zero(const tc_zero_item (&item)[TC_ZERO_MAX], hipStream_t s);

// Stable LSD radix sort on the low `bits` bits of the keys (8-bit digits).
// The sorted data ends in *keys / *vals: the pointers are swapped with the
// tmp pointers when the pass count is odd, so callers free both buffers.
tc_status tc_sort_u64(uint64_t **keys, uint64_t **tmp_keys, int64_t n, int bits, hipStream_t s);
// keys from src (left unchanged), values the input positions 0..n-1: the
// stable sorting permutation of src; the result is in *keys / *vals
tc_status tc_sort_u32_index(const uint32_t *src, uint32_t **keys, uint32_t **vals,
                            uint32_t **tmp_keys, uint32_t **tmp_vals, int64_t n, int bits,
                            hipStream_t s);
// One stable pass: the (key, value) pairs ordered by the 8-bit digit
// (key >> shift) & 255, written to keys_out / vals_out (inputs unchanged).
tc_status tc_partition_u32_u32(const uint32_t *keys, const uint32_t *vals, uint32_t *keys_out,
                               uint32_t *vals_out, int64_t n, int shift, hipStream_t s);
// the same with 64-bit values (hi[i] << 32) | i
tc_status tc_sort_u32_index_hi(const uint32_t *src, const uint32_t *hi, uint32_t **keys,
                               uint64_t **vals, uint32_t **tmp_keys, uint64_t **tmp_vals,
                               int64_t n, int bits, hipStream_t s);
tc_status tc_sort_u64_u32(uint64_t **keys, uint32_t **vals, uint64_t **tmp_keys,
                          uint32_t **tmp_vals, int64_t n, int bits, hipStream_t s);

// ---------------------------------------------------------------------------
// The core: the vertices of the N highest ranks, whose inner triangles the
// middle-pivot count takes from matrix products (tc_core.hip).
// ---------------------------------------------------------------------------
constexpr int TC_CORE_SIZES = 8;
// multiples of 1024 (whole panels of tiles)
__host__ __device__ __forceinline__ int32_t tc_core_ranks(int j) {
    constexpr int32_t K[TC_CORE_SIZES] = {2, 4, 6, 8, 12, 16, 24, 32};
    return K[j] * 1024;
}

// What the scan leaves out: the pairs of core vertex v from end[v - r0] on.
struct tc_core {
    int32_t r0 = 0x7FFFFFFF;  // the core's first rank (no core: above every rank)
    const int64_t *end = nullptr;
};

// The end of pivot v's pairs.
__device__ __forceinline__ int64_t tc_pairs_end(const int64_t *__restrict__ in_ptr, tc_core core,
                                                int64_t v) {
    return v >= core.r0 ? core.end[v - core.r0] : in_ptr[v + 1];
}

// Edges that the orientation samples for the triangles per edge, from this many
// edges on (tc_build.hip).  The sampled sum of at most 127 a sample is within 4%
// of its mean where an edge has ten triangles.
constexpr int TC_SAMPLES = 4096;
constexpr int64_t TC_SAMPLE_MIN_EDGES = 200000;

// ---------------------------------------------------------------------------
// The graph handle.
// ---------------------------------------------------------------------------
struct tc_graph {
    int device = 0;
    int32_t n = 0;           // vertices (sum over a batch)
    int64_t m = 0;           // canonical edges after normalisation
    int32_t num_graphs = 1;  // 1 unless built by tc_batch_create
    int bits = 1;            // bits per vertex id in packed keys
    hipStream_t last_stream = nullptr;
    bool computed = false;
    int32_t status = TC_OK;

    // canonical edges, lexicographic
    int32_t *eu = nullptr, *ev = nullptr;           // [m]
    // symmetric CSR in original ids, rows sorted by id
    int64_t *row_ptr = nullptr;                     // [n+1]
    int32_t *col = nullptr;                         // [2m] (filled on demand)
    uint32_t *sym2e = nullptr;                      // [2m] canonical edge of each slot
    // kept from the build so that col / sym2e can be filled on demand: the
    // first canonical edge whose smaller end is v
    uint32_t *run_us = nullptr;                     // [n]
    // the canonical edges ordered by their larger end (key = ev, val =
    // edge): from the build to the orientation, and on to the symmetric
    // fill unless the middle-pivot count releases them first
    uint32_t *lt_key = nullptr, *lt_val = nullptr;  // [m]
    // degree order: perm[r] = vertex of rank r, rank[v]
    int32_t *rank = nullptr, *perm = nullptr;       // [n]
    // oriented CSR over ranks: row r holds the ranks above r, ascending
    int64_t *orp = nullptr;                         // [n+1]
    int32_t *ocol = nullptr;                        // [m]
    // ocol for the pivots among the top 2^16 ranks: entries at or above
    // rank16_base, less rank16_base (16 bits); other entries read 0
    uint16_t *ocol16 = nullptr;                     // [m + TC_OCOL_PAD, rounded up to even]
    int32_t rank16_base = 0;
    uint32_t *o2e = nullptr;                        // [m] canonical edge of each oriented slot
    int32_t *orow = nullptr;                        // [m] row (rank) of each oriented slot
    // transposed orientation (middle-pivot counting): pairs grouped by the
    // higher end v, entry = (u << 32) | slot of v in N_H(u)
    int64_t *in_ptr = nullptr;                      // [n+1]
    uint64_t *in_pair = nullptr;                    // [m]
    // per-row triangular bit matrices of the middle-pivot scan
    int64_t *rowbase = nullptr;                     // [n+1] first word of each row's matrix
    uint32_t *hitbits = nullptr;                    // [bit_words]
    uint4 *rowinfo = nullptr;                       // [n] rowbase (low, high), row start, row end
    int64_t bit_words = 0;
    // results
    uint32_t *osup = nullptr;                       // [m] support per oriented slot
    uint32_t *esup = nullptr;                       // [m] support per canonical edge
    uint8_t *flag = nullptr;                        // [2m] slot edge has support > 0
    uint64_t *tri = nullptr, *num = nullptr;        // [n]
    double *tcv = nullptr;                          // [n]
    uint64_t *triG = nullptr;                       // [num_graphs]
    // batch bookkeeping (device copies + host copies)
    int64_t *vtx_off = nullptr;                     // device [G+1]
    int64_t *h_vtx_off = nullptr;                   // host [G+1]
    int64_t *h_edge_off = nullptr;                  // host [G+1]
    bool rank_by_graph = false;                     // a graph's ranks are consecutive
    int32_t max_dplus = 0;
    int32_t max_degree = 0;
    // oriented wedges of the rows of the tc_core_ranks(j) highest ranks, the
    // sizes of the core that tc_core.hip takes
    unsigned long long core_wedges[TC_CORE_SIZES] = {};
    int32_t core_n = 0;  // the last count's core
    // triangles per edge, from a sample (0 below TC_SAMPLE_MIN_EDGES)
    double tri_per_edge = 0.0;
    uint32_t *err = nullptr;  // device words: error bits, largest degree, 2 unused

    size_t bytes = 0;  // device bytes held

    // bins of the last count: light 2..light_max, heavy ..huge_min-1, huge
    int32_t light_max = 0, huge_min = 0;
    int32_t algo_used = 0;
    bool slots_used = false;  // the last count merged slots (tc_slots.hip)
    bool single = false;      // built by one workgroup (tc_single.hip)

    // profiling marks (see tc_prof_mark)
    bool prof = false;
    bool prof_build = false, prof_compute = false;
    hipEvent_t prof_ev[TC_PROF_MARKS] = {};
};

// Profiling marks: 0 build start, 1 CSR built, 2 ranked, 3 oriented,
// 4 compute start, 5 binned, 6 light counted, 7 heavy counted,
// 8 huge counted, 9 folded, 10 tri/triG done, 11 aggregated.
bool tc_profiling_on();
void tc_prof_mark(tc_graph *g, int idx, hipStream_t s);

// Pipeline stages (tc_build.hip, tc_count.hip, tc_aggregate.hip).
// Canonical edges from pairs (sorted and deduplicated), or, with simple_rp
// given, from a simple sorted CSR of P entries (simple_rp / simple_col,
// device): the entries above the diagonal, taken in order.
tc_status tc_build_from_pairs(tc_graph *g, const int32_t *d_src, const int32_t *d_dst,
                              int64_t P, const int64_t *d_pair_vtx_base,
                              const int64_t *d_pair_off, int32_t num_graphs, hipStream_t s,
                              const int64_t *simple_rp = nullptr,
                              const int32_t *simple_col = nullptr);
tc_status tc_orient(tc_graph *g, hipStream_t s);
tc_status tc_count(tc_graph *g, const tc_tuning *t, hipStream_t s);
tc_status tc_aggregate(tc_graph *g, hipStream_t s);
// Fills the symmetric adjacency col / sym2e from what the build kept
// (once per handle; no-op when filled).  tc_build.hip.
tc_status tc_ensure_symmetric(tc_graph *g, hipStream_t s);
// Frees lt_key / lt_val (no-op when gone).  tc_build.hip.
void tc_release_transposition(tc_graph *g, hipStream_t s);
tc_status tc_alg_numerator(const tc_graph *g, uint64_t *d_num, hipStream_t s);  // tc_algebraic.hip
// The k <= TOPK_SELECT_MAX largest of tcv[n] (ties by smaller index) into host
// arrays; *found is false, and nothing is written, when more than TOPK_CAP
// values tie around the k-th.  Waits for the stream.  tc_topk.hip.
constexpr uint32_t TOPK_CAP = 4096;
constexpr int32_t TOPK_SELECT_MAX = 1024;
tc_status tc_topk_select(const double *tcv, int32_t n, int32_t k, int32_t *h_verts, double *h_vals,
                         bool *found, hipStream_t s);
tc_status tc_work_stats(tc_graph *g, int64_t *stats, hipStream_t s);
// tc_tuning's default of light_bitmap_pairs, which stands for no choice
constexpr int32_t TC_LIGHT_BITMAP_PAIRS = 64;
tc_status tc_mid_prepare(tc_graph *g, hipStream_t s, bool keep_order = false);
// Takes all its memory before it counts: after TC_ERR_BUDGET or TC_ERR_OOM
// g->osup and *found are as they were.
tc_status tc_count_mid(tc_graph *g, const tc_tuning &t, int lds_limit, int max_entries,
                       unsigned long long *found, hipStream_t s);
// The slot merge (tc_slots.hip) up to this longest oriented row: a slot's merge
// grows with the rows, a table or bitmap lookup does not.  Whole calls, merge
// against the forms above (us): BA attach 32, 0.65 M edges, longest row 50:
// 625 / 853; BA attach 64, 12.9 M edges, 94: 4305 / 5726; R-MAT scale 13, 103:
// 570 / 634; BA attach 100, 126: 1203 / 1175; R-MAT scale 15, 192: 1146 / 931;
// scale 16, 246: 1879 / 955.
constexpr int TC_SLOTS_MAX_DPLUS = 128;
// Graphs for which tc_compute_bytes promises that AUTO stays within the low
// pivot's bound.  AUTO still takes the middle pivot there where all its arrays fit
// into that bound (tc_mid_most_bytes); and where a memory limit leaves no room for
// them it counts with the low pivot, so the order by larger end, which that needs,
// is kept until they are all there.  A larger graph gets the limit's error.
static inline bool tc_low_bytes_promised(const tc_graph *g) {
    return g->m < 600000 || (g->m < 3000000 && g->max_dplus < 32);
}
// The bytes of every block that AUTO's middle pivot and its aggregation allocate,
// as if none were used twice, up to a bound of the bit matrices' size.
int64_t tc_mid_most_bytes(const tc_graph *g);
// Frees what the middle pivot keeps on the handle.
void tc_mid_release(tc_graph *g, hipStream_t s);
// Has what the aggregation after it will allocate: the results on the handle, the
// scratch given back at once for it to take again (tc_aggregate.hip).
tc_status tc_rank_room(tc_graph *g, hipStream_t s);
// Whether AUTO counts in another form where the middle pivot finds no memory.
static inline bool tc_mid_may_yield(const tc_graph *g, const tc_tuning &t) {
    return t.algorithm == TC_ALGO_AUTO &&
           (g->max_dplus <= TC_SLOTS_MAX_DPLUS || tc_low_bytes_promised(g));
}
static inline bool tc_no_memory(tc_status st) { return st == TC_ERR_BUDGET || st == TC_ERR_OOM; }
// tc_core.hip: the core's size for this graph (0: none); its matrix
// (N * N / 32 words of 16 bytes) and the ends of its pairs; its products added
// to g->osup and its triangles to *found (sum: a scratch word).
int32_t tc_core_size(const tc_graph *g);
tc_status tc_core_fill(const tc_graph *g, int32_t N, int64_t *end, uint4 *mat, hipStream_t s);
tc_status tc_core_count(const tc_graph *g, int32_t N, const uint4 *mat, unsigned long long *sum,
                        unsigned long long *found, hipStream_t s);
// One small graph by one workgroup (tc_single.hip): everything that
// tc_build_from_pairs and tc_orient leave but the order by larger ends (made
// again where a consumer needs it), and everything that tc_count and
// tc_aggregate leave.
bool tc_single_fits(int64_t P, int32_t n);
tc_status tc_single_build(tc_graph *g, const int32_t *d_src, const int32_t *d_dst, int64_t P,
                          hipStream_t s);
tc_status tc_single_count(tc_graph *g, hipStream_t s);
// Flat graphs (tc_slots.hip): support per slot into the zeroed g->osup, then
// everything that tc_aggregate fills.
tc_status tc_count_slots(tc_graph *g, unsigned long long *found, hipStream_t s);
tc_status tc_aggregate_slots(tc_graph *g, hipStream_t s);
tc_status tc_mid_stats(tc_graph *g, unsigned long long *acc, hipStream_t s);
// Words of the middle pivot's bit matrices, Σ_r Σ_{t<|N_H(r)|} ceil(t/32)
// (device reduction and one read-back; the stored total once they exist).
tc_status tc_mid_bit_words(const tc_graph *g, int64_t *words, hipStream_t s);
// Upper bound of the device bytes tc_count + tc_aggregate allocate beyond
// what g holds, for the pivot form the tuning (or AUTO) picks.
tc_status tc_count_bytes(tc_graph *g, const tc_tuning *tuning, hipStream_t s, int64_t *bytes);

template <typename T>
tc_status tc_graph_alloc(tc_graph *g, T **p, int64_t count, hipStream_t s) {
    tc_status st = tc_alloc(p, count, s);
    if (st == TC_OK) g->bytes += (size_t)(count > 0 ? count : 1) * sizeof(T);
    return st;
}

// The handle takes p, count entries allocated in tmp, as *slot.  For arrays that
// are made once per handle: only when nothing can fail before they are filled, as
// a later call takes an array that is there as filled.
template <typename T>
void tc_graph_take(tc_graph *g, T **slot, T *p, int64_t count, tc_scratch &tmp) {
    tmp.exchange(p, nullptr);
    *slot = p;
    g->bytes += (size_t)(count > 0 ? count : 1) * sizeof(T);
}

// ---------------------------------------------------------------------------
// Device-side helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ int tc_lane() { return __lane_id(); }

__device__ __forceinline__ uint64_t tc_lanemask_lt() {
    int l = __lane_id();
    return l == 0 ? 0ull : (~0ull >> (64 - l));
}

template <typename T>
__device__ __forceinline__ T tc_wave_sum(T x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, TC_WAVE);
    return x;
}

// Maximum across the 64 lanes of a wavefront.
template <typename T>
__device__ __forceinline__ T tc_wave_max(T x) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        T y = __shfl_xor(x, off, TC_WAVE);
        x = y > x ? y : x;
    }
    return x;
}

// The graph of global vertex id (or, as a graph's ranks take the places of its
// vertices, rank) v: the last g with vtx_off[g] <= v.
__device__ __forceinline__ int32_t tc_graph_of(const int64_t *__restrict__ vtx_off, int32_t G,
                                               int64_t v) {
    int32_t lo = 0, hi = G - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (vtx_off[mid] <= v) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Reserves c places for each thread of a BLOCK-thread workgroup behind the
// counter *count, with one atomic for the workgroup (one per thread or
// wavefront on a shared word serialises: 11 ns each); returns the thread's
// first place.  Every thread calls.  lds: BLOCK / 64 + 1 words.
template <int BLOCK>
__device__ __forceinline__ uint32_t tc_block_reserve(uint32_t c, uint32_t *count, uint32_t *lds);

// Inclusive scan across the 64 lanes of a wavefront.
template <typename T>
__device__ __forceinline__ T tc_wave_incl_scan(T x) {
    int l = __lane_id();
#pragma unroll
    for (int off = 1; off < TC_WAVE; off <<= 1) {
        T y = __shfl_up(x, off, TC_WAVE);
        if (l >= off) x += y;
    }
    return x;
}

template <int BLOCK>
__device__ __forceinline__ uint32_t tc_block_reserve(uint32_t c, uint32_t *count, uint32_t *lds) {
    constexpr int W = BLOCK / TC_WAVE;
    const int w = threadIdx.x / TC_WAVE;
    const uint32_t incl = tc_wave_incl_scan(c);
    if (__lane_id() == TC_WAVE - 1) lds[w] = incl;
    __syncthreads();
    uint32_t before = incl - c, all = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const uint32_t x = lds[q];
        before += q < w ? x : 0u;
        all += x;
    }
    if (threadIdx.x == 0) lds[W] = all ? atomicAdd(count, all) : 0u;
    __syncthreads();
    const uint32_t base = lds[W];
    __syncthreads();
    return base + before;
}

// Raises *word to the workgroup's largest x; reads the word first, so that
// most workgroups of a launch do without the atomic.
template <int BLOCK>
__device__ __forceinline__ void tc_block_raise(uint32_t x, uint32_t *word, uint32_t *lds) {
    x = tc_wave_max(x);
    if (__lane_id() == 0) lds[threadIdx.x / TC_WAVE] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < BLOCK / TC_WAVE; ++q) x = lds[q] > x ? lds[q] : x;
        if (x > __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(word, x);
    }
    __syncthreads();
}
