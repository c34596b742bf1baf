// Stands in for the library's internal header where the fused launch
// (tc_fused.hip, tc_small.h) is compiled for the host: the device features of
// hip_cpu.h and those that these two files use beyond them.
#pragma once
#include "hip_cpu.h"

#include <cmath>

#include "tc.h"

inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline int __clz(uint32_t x) { return x ? __builtin_clz(x) : 32; }
inline int __clzll(uint64_t x) { return x ? __builtin_clzll(x) : 64; }
inline int __ffs(int x) { return x ? __builtin_ctz(x) + 1 : 0; }
inline int __ffsll(uint64_t x) { return x ? __builtin_ctzll(x) + 1 : 0; }

inline uint64_t __ballot(bool p) {
    EmuWave &w = *emu_blk->waves[emu_tid / TC_WAVE];
    w.slots[emu_tid % TC_WAVE] = p;
    w.bar.arrive_and_wait();
    uint64_t r = 0;
    for (int i = 0; i < TC_WAVE; ++i) r |= (w.slots[i] & 1) << i;
    w.bar.arrive_and_wait();
    return r;
}
template <typename T> inline T emu_lane(T x, int src) {
    uint64_t u = 0;
    std::memcpy(&u, &x, sizeof(T));
    const uint64_t r = emu_exchange(u, src);
    T o;
    std::memcpy(&o, &r, sizeof(T));
    return o;
}
template <typename T> inline T __shfl(T x, int src, int = TC_WAVE) { return emu_lane(x, src & 63); }
template <typename T> inline T __shfl_down(T x, unsigned d, int = TC_WAVE) {
    const int l = __lane_id();
    return emu_lane(x, l + (int)d < TC_WAVE ? l + (int)d : l);
}

// one word for each of two calls in turn: the next call's is cleared between the
// barriers of this one
extern std::atomic<int> emu_or[2];
extern thread_local int emu_or_turn;
inline int __syncthreads_or(int p) {
    const int i = emu_or_turn;
    emu_or_turn ^= 1;
    if (p) emu_or[i].store(1);
    emu_blk->bar->arrive_and_wait();
    const int r = emu_or[i].load();
    emu_or[i ^ 1].store(0);
    emu_blk->bar->arrive_and_wait();
    return r;
}
// its uses hold the same value in every lane
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __hip_atomic_fetch_add(p, v, order, scope) \
    std::atomic_ref<std::remove_reference_t<decltype(*(p))>>(*(p)).fetch_add(v)
inline double __ddiv_rn(double a, double b) { return a / b; }

inline int64_t tc_div_up(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline uint64_t tc_lanemask_lt() {
    const int l = __lane_id();
    return l == 0 ? 0ull : (~0ull >> (64 - l));
}
template <typename T> T tc_wave_sum(T x) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, TC_WAVE);
    return x;
}
template <typename T> T tc_wave_max(T x) {
    for (int o = 32; o > 0; o >>= 1) {
        const T y = __shfl_xor(x, o, TC_WAVE);
        x = y > x ? y : x;
    }
    return x;
}
template <typename T> T tc_wave_incl_scan(T x) {
    const int l = __lane_id();
    for (int o = 1; o < TC_WAVE; o <<= 1) {
        const T y = __shfl_up(x, o, TC_WAVE);
        if (l >= o) x += y;
    }
    return x;
}
