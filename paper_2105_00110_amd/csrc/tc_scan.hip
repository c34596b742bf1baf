// Device-wide exclusive prefix sum.
//
// Up to ONE_MAX elements one workgroup scans everything: one launch.  Above,
// reduce-then-scan over tiles of TILE = BLOCK*ITEMS elements: one kernel
// reduces every tile, and a second one rescans each tile in LDS and adds the
// sum of the tiles before it, which every workgroup takes from the tile sums
// itself (a few KB out of the L2): two launches.  Only above PARTIAL_MAX tiles
// are the tile sums scanned by a launch of their own first.  Loads and stores
// are coalesced (striped through LDS); each thread scans ITEMS consecutive
// elements.
//
// The graph build makes some twenty scans of mostly under a million elements,
// so their launches cost more than their bytes: three launches and more for
// each of them were 90 of the 206 launches and 0.40 ms of an R-MAT scale-20
// call.
#include "tc_internal.h"

namespace {

struct ZeroArgs {
    uint32_t *p[TC_ZERO_MAX];
    int64_t words[TC_ZERO_MAX];
};

constexpr int SCAN_BLOCK = 256;
constexpr int SCAN_ITEMS = 16;
constexpr int SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;
constexpr int SCAN_WAVES = SCAN_BLOCK / TC_WAVE;
constexpr int ONE_BLOCK = 1024;
constexpr int ONE_ITEMS = 8;
constexpr int64_t ONE_MAX = 2 * ONE_BLOCK * ONE_ITEMS;  // two rounds of one workgroup
constexpr int64_t PARTIAL_MAX = 4096;

template <typename T>
__device__ T block_sum(T x, T *red) {
    x = tc_wave_sum(x);
    int w = threadIdx.x / TC_WAVE;
    if (__lane_id() == 0) red[w] = x;
    __syncthreads();
    T t = 0;
#pragma unroll
    for (int i = 0; i < SCAN_WAVES; ++i) t += red[i];
    return t;
}

template <typename T>
__global__ __launch_bounds__(SCAN_BLOCK) void k_tile_reduce(const T *__restrict__ in, int64_t n,
                                                            T *__restrict__ partial) {
    __shared__ T red[SCAN_WAVES];
    int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    T acc = 0;
#pragma unroll
    for (int it = 0; it < SCAN_ITEMS; ++it) {
        int64_t i = base + it * SCAN_BLOCK + threadIdx.x;
        if (i < n) acc += in[i];
    }
    T t = block_sum(acc, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// Exclusive scan by one workgroup, ONE_BLOCK * ONE_ITEMS elements a round.
template <typename T>
__global__ __launch_bounds__(ONE_BLOCK) void k_scan_one(const T *in, T *out, int64_t n, T *total) {
    constexpr int W = ONE_BLOCK / TC_WAVE;
    __shared__ T wsum[W];
    const int tid = threadIdx.x, w = tid / TC_WAVE;
    T carry = 0;
    for (int64_t base = 0; base < n; base += ONE_BLOCK * ONE_ITEMS) {
        const int64_t i0 = base + (int64_t)tid * ONE_ITEMS;
        T v[ONE_ITEMS], run = 0;
#pragma unroll
        for (int k = 0; k < ONE_ITEMS; ++k) v[k] = i0 + k < n ? in[i0 + k] : (T)0;
#pragma unroll
        for (int k = 0; k < ONE_ITEMS; ++k) {
            const T x = v[k];
            v[k] = run;
            run += x;
        }
        const T incl = tc_wave_incl_scan(run);
        if (__lane_id() == TC_WAVE - 1) wsum[w] = incl;
        __syncthreads();
        T before = carry + incl - run, all = 0;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const T x = wsum[q];
            before += q < w ? x : (T)0;
            all += x;
        }
#pragma unroll
        for (int k = 0; k < ONE_ITEMS; ++k)
            if (i0 + k < n) out[i0 + k] = v[k] + before;
        carry += all;
        __syncthreads();
    }
    if (total != nullptr && tid == 0) *total = carry;
}

// Exclusive scan of one tile.  tile_off holds the tile sums (SUMMED false:
// the workgroup adds those before its own) or their exclusive scan (SUMMED
// true).  The block that owns the last element writes the grand total.
template <typename T, bool SUMMED>
__global__ __launch_bounds__(SCAN_BLOCK) void k_tile_scan(const T *in, T *out, int64_t n,
                                                          const T *__restrict__ tile_off,
                                                          T *total) {
    __shared__ T buf[SCAN_TILE];
    __shared__ T wsum[SCAN_WAVES];
    int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    int tid = threadIdx.x;
#pragma unroll
    for (int it = 0; it < SCAN_ITEMS; ++it) {
        int j = it * SCAN_BLOCK + tid;
        int64_t i = base + j;
        buf[j] = (i < n) ? in[i] : (T)0;
    }
    __syncthreads();
    T v[SCAN_ITEMS];
    T run = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        v[k] = run;
        run += buf[tid * SCAN_ITEMS + k];
    }
    T incl = tc_wave_incl_scan(run);
    int w = tid / TC_WAVE;
    if (__lane_id() == TC_WAVE - 1) wsum[w] = incl;
    __syncthreads();
    T before = incl - run;
    for (int i = 0; i < w; ++i) before += wsum[i];
    if constexpr (SUMMED) {
        before += tile_off[blockIdx.x];
    } else {
        T acc = 0;
        for (unsigned i = tid; i < blockIdx.x; i += SCAN_BLOCK) acc += tile_off[i];
        __shared__ T red[SCAN_WAVES];
        before += block_sum(acc, red);
    }
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) buf[tid * SCAN_ITEMS + k] = v[k] + before;
    if (total != nullptr && tid == SCAN_BLOCK - 1 && base + SCAN_TILE >= n) {
        *total = before + run;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < SCAN_ITEMS; ++it) {
        int j = it * SCAN_BLOCK + tid;
        int64_t i = base + j;
        if (i < n) out[i] = buf[j];
    }
}

template <typename T>
__global__ void k_set_zero(T *p) { *p = 0; }

template <typename T>
tc_status scan_impl(const T *in, T *out, int64_t n, T *total, hipStream_t s) {
    if (n < 0) return TC_ERR_INVALID_ARG;
    if (n == 0) {
        if (total) {
            k_set_zero<T><<<1, 1, 0, s>>>(total);
            TC_LAUNCHED();
        }
        return TC_OK;
    }
    if (n <= ONE_MAX) {
        k_scan_one<T><<<1, ONE_BLOCK, 0, s>>>(in, out, n, total);
        TC_LAUNCHED();
        return TC_OK;
    }
    int64_t tiles = tc_div_up(n, SCAN_TILE);
    if (tiles > 0x7FFFFFFF) return TC_ERR_UNSUPPORTED;
    tc_scratch tmp(s);
    T *partial = nullptr;
    TC_TRY(tmp.get(&partial, tiles));
    k_tile_reduce<T><<<(unsigned)tiles, SCAN_BLOCK, 0, s>>>(in, n, partial);
    TC_LAUNCHED();
    if (tiles <= PARTIAL_MAX) {
        k_tile_scan<T, false><<<(unsigned)tiles, SCAN_BLOCK, 0, s>>>(in, out, n, partial, total);
    } else {
        TC_TRY(scan_impl<T>(partial, partial, tiles, (T *)nullptr, s));
        k_tile_scan<T, true><<<(unsigned)tiles, SCAN_BLOCK, 0, s>>>(in, out, n, partial, total);
    }
    TC_LAUNCHED();
    return TC_OK;
}

// Each array in turn by the whole grid: 16 bytes a store from its first word on
// where that is aligned, single words for the rest.
__global__ __launch_bounds__(256) void k_zero(ZeroArgs a) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
#pragma unroll
    for (int k = 0; k < TC_ZERO_MAX; ++k) {
        uint32_t *const p = a.p[k];
        const int64_t words = a.words[k];
        const int64_t quads = (reinterpret_cast<uintptr_t>(p) & 15) == 0 ? words / 4 : 0;
        for (int64_t i = t; i < quads; i += step)
            reinterpret_cast<uint4 *>(p)[i] = make_uint4(0u, 0u, 0u, 0u);
        for (int64_t i = 4 * quads + t; i < words; i += step) p[i] = 0u;
    }
}

}  // namespace

tc_status tc_zero(const tc_zero_item (&item)[TC_ZERO_MAX], hipStream_t s) {
    ZeroArgs a = {};
    int64_t all = 0;
    for (int k = 0; k < TC_ZERO_MAX; ++k) {
        a.p[k] = static_cast<uint32_t *>(item[k].p);
        a.words[k] = item[k].p ? item[k].words : 0;
        all += a.words[k];
    }
    const int64_t want = tc_div_up(all, 4 * 256);
    k_zero<<<(unsigned)(want < 1 ? 1 : (want < 2048 ? want : 2048)), 256, 0, s>>>(a);
    TC_LAUNCHED();
    return TC_OK;
}

tc_status tc_scan_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *total,
                      hipStream_t s) {
    return scan_impl<uint32_t>(in, out, n, total, s);
}

tc_status tc_scan_i64(const int64_t *in, int64_t *out, int64_t n, int64_t *total,
                      hipStream_t s) {
    return scan_impl<int64_t>(in, out, n, total, s);
}
