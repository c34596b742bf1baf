// Stable LSD radix sort, 8-bit digits, for the graph build.
//
// Per digit pass (reduce-then-scan form):
//   k_radix_hist    each tile of TILE keys counts its 256 digits in LDS and
//                   writes them digit-major: counts[d * tiles + tile];
//   k_radix_rows    one workgroup per digit scans the digit's counts over
//                   the tiles and keeps their total; with the totals of the
//                   smaller digits this gives, for every (digit, tile), the
//                   first output position of that tile's keys with that
//                   digit (smaller digits first, then earlier tiles: this
//                   is what makes the pass stable).  Up to FEW_TILES tiles
//                   there is no such launch: the counts are written
//                   tile-major and every workgroup of the scatter sums the
//                   few rows before its own (a general scan of the counts
//                   took two to five launches);
//   k_radix_scatter every wavefront ranks its keys with 8 ballots per item
//                   (lanes holding the same digit form a 64-bit peer mask;
//                   the rank is the popcount of lower peers plus the
//                   wavefront's running count of that digit), wavefronts
//                   are combined by a per-digit prefix over the block, and
//                   keys (and values) are written to their final place.
// Tile element order is (wavefront, item, lane), which equals memory order,
// so equal digits keep their input order.
#include "tc_internal.h"

namespace {

constexpr int RB = 8;
constexpr int RADIX = 1 << RB;
// Shape of the big tiles: 8192 elements of up to 8 bytes (key and value) by 512
// threads, 4096 of wider ones by 256; bigger tiles mean longer runs per digit
// in the scatter's stores.  With 512 threads two workgroups of a CU keep 16
// wavefronts resident under the same LDS (256 threads: 8, and twice the
// registers); 5 M 8-byte keys 36 -> 31 us a pass, 2^28 of them 1.34 -> 1.27 ms
// (1024 threads: 1.5 ms).  Wider elements are staged in two rounds (keys, then
// values, through the same LDS buffer), which keeps their LDS near 43 KB and
// three workgroups resident; 512 threads made their pass slower (2.25 against
// 2.13 ms for 2.6e8).
template <typename K, typename V, bool HAS_VAL>
constexpr bool sort_wide() {
    return sizeof(K) + (HAS_VAL ? sizeof(V) : 0) > 8;
}
template <typename K, typename V, bool HAS_VAL>
constexpr int sort_block() {
    return sort_wide<K, V, HAS_VAL>() ? 256 : 512;
}
constexpr int BIG_ITEMS = 16;
// Below this many elements the big tiles would leave CUs idle: tiles of 2048,
// 256 threads of 8 elements.
constexpr int64_t SORT_BIG_TILES_MIN = (int64_t)1 << 22;
constexpr int SMALL_BLOCK = 256;
constexpr int SORT_SMALL_ITEMS = 8;
// Up to this many tiles the scatter sums the tile counts itself: at 128 tiles
// (2^18 keys) that is 128 KB out of the L2 per workgroup, about the time of
// the launch that it saves.
constexpr int64_t FEW_TILES = 128;

static_assert(SMALL_BLOCK >= RADIX, "one digit per thread in the digit scans");

struct NoVal {};

// Lane l counts in copy l mod COPIES, so that lanes with one digit (skewed ids, the
// upper digits of degrees or of ids in order) meet at an address COPIES times
// less often; the copies of a digit lie in banks of their own.  With a copy per
// wavefront instead: 3.4e7 ids of R-MAT edges 93 us, 63 so; 1.7e7 degrees 57, 23;
// no change on uniform keys.
constexpr int COPIES = 8;

template <typename K, int SORT_BLOCK, int SORT_ITEMS, bool FEW>
__global__ __launch_bounds__(SORT_BLOCK) void k_radix_hist(const K *__restrict__ keys, int64_t n,
                                                           int shift, uint32_t *__restrict__ counts,
                                                           int64_t tiles) {
    constexpr int SORT_TILE = SORT_BLOCK * SORT_ITEMS;
    __shared__ uint32_t hist[RADIX][COPIES];
    for (int i = threadIdx.x; i < RADIX * COPIES; i += SORT_BLOCK) (&hist[0][0])[i] = 0;
    __syncthreads();
    const int copy = threadIdx.x % COPIES;
    const int64_t base = (int64_t)blockIdx.x * SORT_TILE;
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; ++it) {
        const int64_t i = base + it * SORT_BLOCK + threadIdx.x;
        if (i < n) atomicAdd(&hist[(uint32_t)(keys[i] >> shift) & (RADIX - 1)][copy], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < RADIX; d += SORT_BLOCK) {
        uint32_t c = 0;
#pragma unroll
        for (int q = 0; q < COPIES; ++q) c += hist[d][q];
        if constexpr (FEW) counts[(int64_t)blockIdx.x * RADIX + d] = c;
        else counts[(int64_t)d * tiles + blockIdx.x] = c;
    }
}

// Exclusive scan of one digit's counts over the tiles, in place; tot[digit] =
// their sum.  Bound by the round trip of a round (4 KB a workgroup), so a
// thread takes four counts at a time.
constexpr int ROWS_BLOCK = 1024;
constexpr int ROWS_ITEMS = 4;

__global__ __launch_bounds__(ROWS_BLOCK) void k_radix_rows(uint32_t *__restrict__ counts,
                                                           int64_t tiles,
                                                           uint32_t *__restrict__ tot) {
    constexpr int W = ROWS_BLOCK / TC_WAVE;
    __shared__ uint32_t wsum[W];
    uint32_t *row = counts + (int64_t)blockIdx.x * tiles;
    const int tid = threadIdx.x, w = tid / TC_WAVE;
    uint32_t carry = 0;
    for (int64_t base = 0; base < tiles; base += ROWS_BLOCK * ROWS_ITEMS) {
        const int64_t i0 = base + (int64_t)tid * ROWS_ITEMS;
        uint32_t v[ROWS_ITEMS], run = 0;
#pragma unroll
        for (int k = 0; k < ROWS_ITEMS; ++k) v[k] = i0 + k < tiles ? row[i0 + k] : 0u;
#pragma unroll
        for (int k = 0; k < ROWS_ITEMS; ++k) {
            const uint32_t x = v[k];
            v[k] = run;
            run += x;
        }
        const uint32_t incl = tc_wave_incl_scan(run);
        if (__lane_id() == TC_WAVE - 1) wsum[w] = incl;
        __syncthreads();
        uint32_t before = carry + incl - run, all = 0;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const uint32_t x = wsum[q];
            before += q < w ? x : 0u;
            all += x;
        }
#pragma unroll
        for (int k = 0; k < ROWS_ITEMS; ++k)
            if (i0 + k < tiles) row[i0 + k] = v[k] + before;
        carry += all;
        __syncthreads();
    }
    if (tid == 0) tot[blockIdx.x] = carry;
}

// Exclusive scan of one value per digit (the first RADIX threads; the others
// pass 0).
__device__ __forceinline__ uint32_t digit_scan(uint32_t x, uint32_t *wsum) {
    const int w = threadIdx.x / TC_WAVE;
    const uint32_t incl = tc_wave_incl_scan(x);
    if (__lane_id() == TC_WAVE - 1) wsum[w] = incl;
    __syncthreads();
    uint32_t before = incl - x;
    for (int q = 0; q < w; ++q) before += wsum[q];
    __syncthreads();
    return before;
}

template <typename K, typename V, bool HAS_VAL, int SORT_BLOCK, int SORT_ITEMS, bool FEW>
__global__ __launch_bounds__(SORT_BLOCK) void k_radix_scatter(
    const K *__restrict__ kin, const V *__restrict__ vin, K *__restrict__ kout,
    V *__restrict__ vout, int64_t n, int shift, const uint32_t *__restrict__ counts,
    int64_t tiles, const uint32_t *__restrict__ tot, const uint32_t *__restrict__ vhi) {
    constexpr int SORT_TILE = SORT_BLOCK * SORT_ITEMS;
    constexpr int SORT_WAVES = SORT_BLOCK / TC_WAVE;
    // The tile is first put in digit order in LDS, then written out by
    // consecutive threads to consecutive positions of each digit's run, so
    // the global stores coalesce.
    __shared__ uint32_t wcnt[SORT_WAVES][RADIX];
    __shared__ uint32_t gbase[RADIX];   // global start of the tile's keys of each digit
    __shared__ uint32_t lbase[RADIX];   // start of each digit within the tile
    constexpr int KB = sizeof(K), VB = HAS_VAL ? sizeof(V) : 0;
    constexpr bool SPLIT = HAS_VAL && KB + VB > 8;  // keys and values staged in turn
    constexpr int STAGE = SORT_TILE * (SPLIT ? (KB > VB ? KB : VB) : KB + VB);
    __shared__ __align__(16) unsigned char sraw[STAGE];
    __shared__ uint8_t sdig[SPLIT ? SORT_TILE : 1];  // digit of each staged position
    K *skey = reinterpret_cast<K *>(sraw);
    V *sval = reinterpret_cast<V *>(SPLIT ? sraw : sraw + (size_t)SORT_TILE * KB);
    for (int i = threadIdx.x; i < SORT_WAVES * RADIX; i += SORT_BLOCK) (&wcnt[0][0])[i] = 0;
    __syncthreads();

    const int w = threadIdx.x / TC_WAVE;
    const int lane = __lane_id();
    const uint64_t lt = tc_lanemask_lt();
    const int64_t tbase = (int64_t)blockIdx.x * SORT_TILE;
    const int64_t wbase = tbase + (int64_t)w * (TC_WAVE * SORT_ITEMS);
    const int tn = (int)((n - tbase) < SORT_TILE ? (n - tbase) : SORT_TILE);

    K key[SORT_ITEMS];
    V val[SORT_ITEMS];
    uint32_t rnk[SORT_ITEMS];
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; ++it) {
        int64_t i = wbase + it * TC_WAVE + lane;
        bool valid = i < n;
        key[it] = valid ? kin[i] : (K)0;
        // no value array: the value is the element's index, with vhi[i] in
        // the high half for 64-bit values when vhi is given
        if constexpr (HAS_VAL) {
            V v = 0;
            if (valid) {
                if (vin) {
                    v = vin[i];
                } else {
                    v = (V)i;
                    if constexpr (sizeof(V) == 8)
                        if (vhi) v |= (V)vhi[i] << 32;
                }
            }
            val[it] = v;
        }
    }
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; ++it) {
        int64_t i = wbase + it * TC_WAVE + lane;
        bool valid = i < n;
        uint32_t d = (uint32_t)(key[it] >> shift) & (RADIX - 1);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            bool bit = (d >> b) & 1u;
            uint64_t bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        uint32_t prior = 0;
        if (valid) prior = wcnt[w][d];
        rnk[it] = prior + (uint32_t)__popcll(peers & lt);
        // the highest peer publishes the new running count of this digit
        bool last = valid && ((peers >> lane) == 1ull);
        if (last) wcnt[w][d] = prior + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    // per digit: offsets of the waves, the tile total, and the global base
    {
        __shared__ uint32_t wsum[SORT_WAVES];
        const int d = threadIdx.x;
        const bool own = d < RADIX;
        uint32_t tile_tot = 0;
        if (own) {
#pragma unroll
            for (int q = 0; q < SORT_WAVES; ++q) {
                uint32_t c = wcnt[q][d];
                wcnt[q][d] = tile_tot;
                tile_tot += c;
            }
        }
        // keys of this digit in all tiles, and in those before this one
        uint32_t all = 0, before = 0;
        if constexpr (FEW) {
            const int nt = (int)tiles;
            if (own) {
#pragma unroll 16
                for (int t = 0; t < nt; ++t) {
                    const uint32_t c = counts[t * RADIX + d];
                    all += c;
                    before += t < (int)blockIdx.x ? c : 0u;
                }
            }
        } else if (own) {
            all = tot[d];
            before = counts[(int64_t)d * tiles + blockIdx.x];
        }
        const uint32_t gb = digit_scan(all, wsum) + before;
        // start of the digit within the tile
        const uint32_t lb = digit_scan(tile_tot, wsum);
        if (own) {
            gbase[d] = gb;
            lbase[d] = lb;
        }
    }
    __syncthreads();
    // place of each item in the tile's digit order
#pragma unroll
    for (int it = 0; it < SORT_ITEMS; ++it) {
        int64_t i = wbase + it * TC_WAVE + lane;
        if (i < n) {
            uint32_t d = (uint32_t)(key[it] >> shift) & (RADIX - 1);
            rnk[it] += lbase[d] + wcnt[w][d];
            skey[rnk[it]] = key[it];
            if constexpr (SPLIT) sdig[rnk[it]] = (uint8_t)d;
            else if constexpr (HAS_VAL) sval[rnk[it]] = val[it];
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < tn; j += SORT_BLOCK) {
        const K k = skey[j];
        const uint32_t d = (uint32_t)(k >> shift) & (RADIX - 1);
        const uint32_t pos = gbase[d] + (uint32_t)j - lbase[d];
        kout[pos] = k;
        if constexpr (HAS_VAL && !SPLIT) vout[pos] = sval[j];
    }
    if constexpr (SPLIT) {
        __syncthreads();
#pragma unroll
        for (int it = 0; it < SORT_ITEMS; ++it) {
            int64_t i = wbase + it * TC_WAVE + lane;
            if (i < n) sval[rnk[it]] = val[it];
        }
        __syncthreads();
        for (int j = threadIdx.x; j < tn; j += SORT_BLOCK) {
            const uint32_t d = sdig[j];
            vout[gbase[d] + (uint32_t)j - lbase[d]] = sval[j];
        }
    }
}

// counts: tiles * RADIX words, then the RADIX digit totals
template <typename K, typename V, bool HAS_VAL, int BLOCK, int ITEMS, bool FEW>
tc_status radix_pass_form(const K *in, const V *vin, K *kout, V *vout, int64_t n, int shift,
                          uint32_t *counts, int64_t tiles, const uint32_t *vhi, hipStream_t s) {
    uint32_t *tot = counts + tiles * RADIX;
    k_radix_hist<K, BLOCK, ITEMS, FEW><<<(unsigned)tiles, BLOCK, 0, s>>>(in, n, shift, counts, tiles);
    TC_LAUNCHED();
    if constexpr (!FEW) {
        k_radix_rows<<<RADIX, ROWS_BLOCK, 0, s>>>(counts, tiles, tot);
        TC_LAUNCHED();
    }
    k_radix_scatter<K, V, HAS_VAL, BLOCK, ITEMS, FEW><<<(unsigned)tiles, BLOCK, 0, s>>>(
        in, vin, kout, vout, n, shift, counts, tiles, tot, vhi);
    TC_LAUNCHED();
    return TC_OK;
}

// One pass of n >= 1 elements; counts holds (tiles + 1) * RADIX words.
template <typename K, typename V, bool HAS_VAL>
tc_status radix_pass(const K *in, const V *vin, K *kout, V *vout, int64_t n, int shift,
                     uint32_t *counts, int64_t tiles, const uint32_t *vhi, hipStream_t s) {
    if (n >= SORT_BIG_TILES_MIN)
        return radix_pass_form<K, V, HAS_VAL, sort_block<K, V, HAS_VAL>(), BIG_ITEMS, false>(
            in, vin, kout, vout, n, shift, counts, tiles, vhi, s);
    if (tiles <= FEW_TILES)
        return radix_pass_form<K, V, HAS_VAL, SMALL_BLOCK, SORT_SMALL_ITEMS, true>(
            in, vin, kout, vout, n, shift, counts, tiles, vhi, s);
    return radix_pass_form<K, V, HAS_VAL, SMALL_BLOCK, SORT_SMALL_ITEMS, false>(
        in, vin, kout, vout, n, shift, counts, tiles, vhi, s);
}

template <typename K, typename V, bool HAS_VAL>
int64_t sort_tiles(int64_t n) {
    return tc_div_up(n, (int64_t)(n >= SORT_BIG_TILES_MIN
                                      ? sort_block<K, V, HAS_VAL>() * BIG_ITEMS
                                      : SMALL_BLOCK * SORT_SMALL_ITEMS));
}

// src, when given, is read by the first pass in place of *keys (which then
// needs no contents); with iota the first pass takes each element's index as
// its value in place of *vals.  *keys and *tkeys are ping-pong buffers as
// usual.  With either, at least one pass runs, so the result is always
// written to the buffers.
template <typename K, typename V, bool HAS_VAL>
tc_status radix_sort(K **keys, V **vals, K **tkeys, V **tvals, int64_t n, int bits, hipStream_t s,
                     const K *src = nullptr, bool iota = false, const uint32_t *vhi = nullptr) {
    if (n < 0 || bits < 0 || bits > (int)(8 * sizeof(K))) return TC_ERR_INVALID_ARG;
    const bool fresh = src != nullptr || iota;
    if (n == 0 || (!fresh && (n <= 1 || bits == 0))) return TC_OK;
    if (fresh && bits == 0) bits = 1;  // keys below 2^0 are all zero: one pass keeps the order
    if (n >= (int64_t)0xFFFFFFFFll) return TC_ERR_UNSUPPORTED;
    const int64_t tiles = sort_tiles<K, V, HAS_VAL>(n);
    tc_scratch tmp(s);
    uint32_t *counts = nullptr;
    TC_TRY(tmp.get(&counts, (tiles + 1) * RADIX));
    for (int shift = 0; shift < bits; shift += RB) {
        const K *in = (src && shift == 0) ? src : *keys;
        const V *vin = (HAS_VAL && !(iota && shift == 0)) ? *vals : nullptr;
        V *vout = HAS_VAL ? *tvals : nullptr;
        const uint32_t *vh = shift == 0 ? vhi : nullptr;
        TC_TRY((radix_pass<K, V, HAS_VAL>(in, vin, *tkeys, vout, n, shift, counts, tiles, vh, s)));
        K *tk = *keys;
        *keys = *tkeys;
        *tkeys = tk;
        if constexpr (HAS_VAL) {
            V *tv = *vals;
            *vals = *tvals;
            *tvals = tv;
        }
    }
    return TC_OK;
}

}  // namespace

tc_status tc_sort_u64(uint64_t **keys, uint64_t **tmp_keys, int64_t n, int bits, hipStream_t s) {
    uint32_t *nv = nullptr, *ntv = nullptr;
    return radix_sort<uint64_t, uint32_t, false>(keys, &nv, tmp_keys, &ntv, n, bits, s);
}


tc_status tc_sort_u32_index(const uint32_t *src, uint32_t **keys, uint32_t **vals,
                            uint32_t **tmp_keys, uint32_t **tmp_vals, int64_t n, int bits,
                            hipStream_t s) {
    return radix_sort<uint32_t, uint32_t, true>(keys, vals, tmp_keys, tmp_vals, n, bits, s, src,
                                                true);
}

tc_status tc_sort_u32_index_hi(const uint32_t *src, const uint32_t *hi, uint32_t **keys,
                               uint64_t **vals, uint32_t **tmp_keys, uint64_t **tmp_vals,
                               int64_t n, int bits, hipStream_t s) {
    return radix_sort<uint32_t, uint64_t, true>(keys, vals, tmp_keys, tmp_vals, n, bits, s, src,
                                                true, hi);
}

tc_status tc_sort_u64_u32(uint64_t **keys, uint32_t **vals, uint64_t **tmp_keys,
                          uint32_t **tmp_vals, int64_t n, int bits, hipStream_t s) {
    return radix_sort<uint64_t, uint32_t, true>(keys, vals, tmp_keys, tmp_vals, n, bits, s);
}

tc_status tc_partition_u32_u32(const uint32_t *keys, const uint32_t *vals, uint32_t *keys_out,
                               uint32_t *vals_out, int64_t n, int shift, hipStream_t s) {
    if (n < 0 || shift < 0 || shift > 24) return TC_ERR_INVALID_ARG;
    if (n == 0) return TC_OK;
    if (n >= (int64_t)0xFFFFFFFFll) return TC_ERR_UNSUPPORTED;
    const int64_t tiles = sort_tiles<uint32_t, uint32_t, true>(n);
    tc_scratch tmp(s);
    uint32_t *counts = nullptr;
    TC_TRY(tmp.get(&counts, (tiles + 1) * RADIX));
    return radix_pass<uint32_t, uint32_t, true>(keys, vals, keys_out, vals_out, n, shift, counts,
                                                tiles, nullptr, s);
}

