// The k best vertices for a caller in host memory, without sorting all n.
//
// Keys are the complements of tc's bit patterns (tc >= 0, so they order like
// the values, largest first); ties go to the smaller id.  Two passes of a
// 13-bit digit histogram narrow the k-th key down to 26 bits (the exponent
// and 14 bits of the mantissa), a third pass collects every key up to that
// prefix, and one workgroup sorts the collected (key, id) pairs in LDS and
// writes the first k.  If more than TOPK_CAP keys share the prefixes up to
// the k-th (values with very many ties, e.g. all zero) nothing is written
// and the caller sorts everything instead.
//
// What bounds it: three reads of tc and five short launches.  At n = 2^20,
// k = 10 (R-MAT scale 20) the 8-pass sort of all keys took 262 us of device
// time; this takes 24 us.
#include <string.h>

#include "tc_internal.h"

namespace {

constexpr int HB = 1024;               // threads of every kernel here
constexpr int DIGIT = 13;
constexpr int BINS = 1 << DIGIT;
constexpr int SHIFT0 = 64 - DIGIT;     // first digit
constexpr int SHIFT1 = 64 - 2 * DIGIT; // second digit
constexpr int PER = BINS / HB;         // bins per thread
constexpr int WAVES = HB / TC_WAVE;

__device__ __forceinline__ uint64_t topk_key(double x) {
    return ~(uint64_t)__double_as_longlong(x);
}

// The bin that holds the need-th smallest key of hist (need >= 1; hist holds
// at least that many) and the keys in the bins before it.  Whole workgroup.
struct Pick {
    uint32_t bin, before, count;
};

__device__ Pick topk_pick(const uint32_t *__restrict__ hist, uint32_t need) {
    __shared__ uint32_t wsum[WAVES];
    __shared__ Pick res;
    const int tid = threadIdx.x, w = tid / TC_WAVE, lane = __lane_id();
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        c[q] = hist[tid * PER + q];
        sum += c[q];
    }
    const uint32_t incl = tc_wave_incl_scan(sum);
    if (lane == TC_WAVE - 1) wsum[w] = incl;
    __syncthreads();
    uint32_t before = incl - sum;
    for (int q = 0; q < w; ++q) before += wsum[q];
    if (before < need && need <= before + sum) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (before < need && need <= before + c[q])
                res = Pick{(uint32_t)(tid * PER + q), before, c[q]};
            before += c[q];
        }
    }
    __syncthreads();
    const Pick r = res;
    __syncthreads();
    return r;
}

// hist[0]: the first digit of every key; hist[1] (SECOND): the second digit
// of the keys in the first digit's picked bin.
template <bool SECOND>
__global__ __launch_bounds__(HB) void k_topk_hist(const double *__restrict__ tcv, int32_t n,
                                                  uint32_t k, uint32_t *__restrict__ hist) {
    __shared__ uint32_t bins[BINS];
    for (int i = threadIdx.x; i < BINS; i += HB) bins[i] = 0;
    uint32_t d0 = 0;
    if constexpr (SECOND) d0 = topk_pick(hist, k).bin;
    __syncthreads();
    for (int64_t v = (int64_t)blockIdx.x * HB + threadIdx.x; v < n; v += (int64_t)gridDim.x * HB) {
        const uint64_t key = topk_key(tcv[v]);
        const uint32_t a = (uint32_t)(key >> SHIFT0);
        if constexpr (SECOND) {
            if (a == d0) atomicAdd(&bins[(uint32_t)(key >> SHIFT1) & (BINS - 1)], 1u);
        } else {
            atomicAdd(&bins[a], 1u);
        }
    }
    __syncthreads();
    uint32_t *out = hist + (SECOND ? BINS : 0);
    for (int i = threadIdx.x; i < BINS; i += HB)
        if (bins[i]) atomicAdd(&out[i], bins[i]);
}

// Every key whose first 26 bits are at most the k-th key's, in any order;
// *count receives how many (TOPK_CAP + 1 or more: not collected).
__global__ __launch_bounds__(HB) void k_topk_collect(const double *__restrict__ tcv, int32_t n,
                                                     uint32_t k, const uint32_t *__restrict__ hist,
                                                     uint32_t *__restrict__ count,
                                                     uint64_t *__restrict__ ckey,
                                                     uint32_t *__restrict__ cid) {
    const Pick p0 = topk_pick(hist, k);
    const Pick p1 = topk_pick(hist + BINS, k - p0.before);
    const uint32_t total = p0.before + p1.before + p1.count;
    if (total > TOPK_CAP) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicMax(count, total);
        return;
    }
    const uint64_t last = ((uint64_t)p0.bin << DIGIT) | p1.bin;
    for (int64_t v = (int64_t)blockIdx.x * HB + threadIdx.x; v < n; v += (int64_t)gridDim.x * HB) {
        const uint64_t key = topk_key(tcv[v]);
        if ((key >> SHIFT1) <= last) {
            const uint32_t at = atomicAdd(count, 1u);  // total <= TOPK_CAP of them
            ckey[at] = key;
            cid[at] = (uint32_t)v;
        }
    }
}

// One workgroup: the collected pairs in order, the first k written.
__global__ __launch_bounds__(HB) void k_topk_final(const uint32_t *__restrict__ count, uint32_t k,
                                                   const uint64_t *__restrict__ ckey,
                                                   const uint32_t *__restrict__ cid,
                                                   const double *__restrict__ tcv,
                                                   int32_t *__restrict__ verts,
                                                   double *__restrict__ vals) {
    __shared__ uint64_t sk[TOPK_CAP];
    __shared__ uint32_t si[TOPK_CAP];
    const uint32_t c = *count;
    if (c > TOPK_CAP) return;
    int P = 1;
    while (P < (int)c) P <<= 1;
    for (int j = threadIdx.x; j < P; j += HB) {
        sk[j] = j < (int)c ? ckey[j] : ~0ull;
        si[j] = j < (int)c ? cid[j] : 0xFFFFFFFFu;
    }
    __syncthreads();
    for (int w = 2; w <= P; w <<= 1) {
        for (int j = w >> 1; j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < (P >> 1); t += HB) {
                const int a = ((t & ~(j - 1)) << 1) | (t & (j - 1)), b = a + j;
                const uint64_t ka = sk[a], kb = sk[b];
                const uint32_t ia = si[a], ib = si[b];
                const bool gt = ka > kb || (ka == kb && ia > ib);
                if (gt == ((a & w) == 0)) {
                    sk[a] = kb;
                    sk[b] = ka;
                    si[a] = ib;
                    si[b] = ia;
                }
            }
            __syncthreads();
        }
    }
    for (uint32_t j = threadIdx.x; j < k; j += HB) {
        verts[j] = (int32_t)si[j];
        vals[j] = tcv[si[j]];
    }
}

}  // namespace

tc_status tc_topk_select(const double *tcv, int32_t n, int32_t k, int32_t *h_verts, double *h_vals,
                         bool *found, hipStream_t s) {
    *found = false;
    tc_scratch tmp(s);
    uint32_t *hist = nullptr;  // the two histograms, then the count
    uint64_t *ckey = nullptr;
    uint32_t *cid = nullptr;
    unsigned char *out = nullptr;  // values, then vertices
    TC_TRY(tmp.get(&hist, 2 * BINS + 1));
    TC_TRY(tmp.get(&ckey, TOPK_CAP));
    TC_TRY(tmp.get(&cid, TOPK_CAP));
    TC_TRY(tmp.get(&out, (int64_t)k * 12));
    uint32_t *count = hist + 2 * BINS;
    double *d_vals = reinterpret_cast<double *>(out);
    int32_t *d_verts = reinterpret_cast<int32_t *>(d_vals + k);
    TC_TRY(tc_zero({{hist, 2 * BINS + 1}}, s));
    // four keys per thread, at most two workgroups per CU
    const int64_t want = tc_div_up(n, 4 * HB);
    const unsigned grid = (unsigned)(want < 512 ? want : 512);
    k_topk_hist<false><<<grid, HB, 0, s>>>(tcv, n, (uint32_t)k, hist);
    TC_LAUNCHED();
    k_topk_hist<true><<<grid, HB, 0, s>>>(tcv, n, (uint32_t)k, hist);
    TC_LAUNCHED();
    k_topk_collect<<<grid, HB, 0, s>>>(tcv, n, (uint32_t)k, hist, count, ckey, cid);
    TC_LAUNCHED();
    k_topk_final<<<1, HB, 0, s>>>(count, (uint32_t)k, ckey, cid, tcv, d_verts, d_vals);
    TC_LAUNCHED();
    uint32_t h_count = 0;
    unsigned char h_out[12 * TOPK_SELECT_MAX];
    TC_HIP(hipMemcpyAsync(&h_count, count, 4, hipMemcpyDeviceToHost, s));
    TC_HIP(hipMemcpyAsync(h_out, out, (size_t)k * 12, hipMemcpyDeviceToHost, s));
    TC_HIP(hipStreamSynchronize(s));
    if (h_count > TOPK_CAP) return TC_OK;
    if (h_vals) memcpy(h_vals, h_out, sizeof(double) * k);
    memcpy(h_verts, h_out + sizeof(double) * k, sizeof(int32_t) * k);
    *found = true;
    return TC_OK;
}
