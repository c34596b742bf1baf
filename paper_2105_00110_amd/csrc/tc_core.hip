// Triangles inside the core, the vertices of the N highest ranks, by matrix
// products.
//
// On a skewed graph the last ranks are densely connected among themselves: at
// R-MAT scale 20 the 8192 highest of 10^6 vertices hold 19% of the edges, a
// density of 9%, and 47% of the oriented wedges that the middle pivot scans.
// For such a block the symmetric 0/1 matrix A is the better form: (A A)(u, v)
// is the number of common neighbours of u and v inside it, so for an edge it
// is what the triangles with all three ends in the core add to its support.
// A triangle lies inside the core exactly if its lowest end does, so the scan
// drops the pairs (u, v) with u in the core (a suffix of every pivot's pair
// list, tc_core::end), the fold the rows u, and this adds the products.
//
// The products run on the matrix cores in the 4-bit format, whose values 0
// and 1 are exact, with 32-bit sums: whole numbers of at most N < 2^24, so
// exact too.  Only the tiles on and above the diagonal are formed: N^3
// operations.
//
// Matrix layout: fragments of 32 rows x 64 columns, 1 KB each, in the order
// in which the lanes of a wavefront hold them as an operand (lane l: row
// l mod 32, the 32 columns of half l / 32, 4 bits each): fragment (kb, R) at
// kb * N/32 + R.  A tile's rows are then consecutive for every kb, a load is
// 16 consecutive bytes per lane, in device memory and in LDS, and both
// operands of a product read the same array.  Which of the 32 columns a
// nibble stands for does not matter, as both operands order them alike.
#include "tc_internal.h"

namespace {

constexpr int CT = 128;             // rows and columns of a tile
constexpr int CK = 128;             // columns of A per step
constexpr int AHEAD = 2;            // steps whose loads are in flight
constexpr int CBLOCK = 256;         // 2 x 2 wavefronts of 64 x 64
constexpr int PANEL = 8;            // tile columns per panel
constexpr int FILL_ROWS = 8;        // rows per workgroup of k_core_fill
constexpr int FRAG = 64;            // 16-byte words of a fragment
constexpr int STEP_WORDS = 2 * (CT / 32) * (CK / 64) * FRAG;  // 16-byte words of one step
static_assert(AHEAD % 2 == 0 && 1024 % (CK * AHEAD) == 0, "whole rounds of steps and stages");
static_assert(2 * STEP_WORDS * 16 >= CT * CT * 2, "the counts of a tile reuse the two stages");

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// 8 bits spread to the low bits of 8 nibbles, as the 4-bit value 1.0 (0b0010).
__device__ __forceinline__ uint32_t nibbles(uint32_t b) {
    b = (b | b << 12) & 0x000F000Fu;
    b = (b | b << 6) & 0x03030303u;
    b = (b | b << 3) & 0x11111111u;
    return b << 1;
}

// The matrix and, per core vertex, the end of its pairs with lower ends below
// the core.  A workgroup takes FILL_ROWS rows, a wavefront each: the higher
// neighbours from the oriented row, the lower ones from the pair list (by
// ascending lower end, so those of the core come last), into a row of bits in
// LDS, which is then spread to nibbles.  Eight rows make 128 consecutive
// bytes of a fragment.  Bound by the store of N^2 / 2 bytes.
__global__ __launch_bounds__(64 * FILL_ROWS) void k_core_fill(
    int32_t r0, int32_t N, const int64_t *__restrict__ orp, const int32_t *__restrict__ ocol,
    const int64_t *__restrict__ in_ptr, const uint64_t *__restrict__ in_pair,
    int64_t *__restrict__ end, uint4 *__restrict__ mat) {
    extern __shared__ uint32_t rows[];
    const int W = N / 32, stride = W + FILL_ROWS;  // the rows' words lie in different banks
    const int w = threadIdx.x / TC_WAVE, lane = __lane_id();
    const int row0 = blockIdx.x * FILL_ROWS;
    uint32_t *bits = rows + w * stride;
    for (int x = lane; x < W; x += TC_WAVE) bits[x] = 0u;
    __syncthreads();
    const int32_t v = r0 + row0 + w;
    for (int64_t k = orp[v] + lane; k < orp[v + 1]; k += TC_WAVE) {
        const int32_t c = ocol[k] - r0;
        atomicOr(&bits[c >> 5], 1u << (c & 31));
    }
    // the first pair whose lower end is in the core: 64 probes per step
    const int64_t stop = in_ptr[v + 1];
    int64_t lo = in_ptr[v], hi = stop;
    while (lo < hi) {
        const int64_t p = lo + (hi - lo) * lane / TC_WAVE;  // ascending, lo first
        const int below = __popcll(__ballot((int32_t)(in_pair[p] >> 32) < r0));
        if (below == 0) break;  // the pair at lo already is
        const int64_t last = lo + (hi - lo) * (below - 1) / TC_WAVE;
        hi = below < TC_WAVE ? lo + (hi - lo) * below / TC_WAVE : hi;
        lo = last + 1;
    }
    if (lane == 0) end[row0 + w] = lo;
    for (int64_t i = lo + lane; i < stop; i += TC_WAVE) {
        const int32_t c = (int32_t)(in_pair[i] >> 32) - r0;
        atomicOr(&bits[c >> 5], 1u << (c & 31));
    }
    __syncthreads();
    const int NR = N / 32;
    for (int t = threadIdx.x; t < W * FILL_ROWS; t += blockDim.x) {
        const int q = t % FILL_ROWS, x = t / FILL_ROWS;
        const int row = row0 + q;
        const uint32_t b = rows[q * stride + x];
        mat[((int64_t)(x >> 1) * NR + (row >> 5)) * FRAG + (row & 31) + 32 * (x & 1)] =
            make_uint4(nibbles(b & 0xFFu), nibbles(b >> 8 & 0xFFu), nibbles(b >> 16 & 0xFFu),
                       nibbles(b >> 24));
    }
}

// Tile number t of the upper triangle: panels of PANEL tile columns, row by
// row inside a panel.
__device__ __forceinline__ void core_tile(int64_t t, int &I, int &J) {
    // tiles before panel p: PANEL^2 p (p - 1) / 2 + PANEL (PANEL + 1) / 2 p
    const auto before = [](int64_t p) {
        return PANEL * PANEL * (p * (p - 1) / 2) + (int64_t)PANEL * (PANEL + 1) / 2 * p;
    };
    int64_t p = 0;
    while (before(p + 1) <= t) ++p;
    int64_t x = t - before(p);
    if (x < (int64_t)PANEL * PANEL * p) {
        I = (int)(x / PANEL);
        J = (int)(PANEL * p + x % PANEL);
        return;
    }
    x -= (int64_t)PANEL * PANEL * p;
    int r = 0;
    while (x >= PANEL - r) x -= PANEL - r++;
    I = (int)(PANEL * p) + r;
    J = I + (int)x;
}

// One tile of A A per workgroup, 64 x 64 of it per wavefront, and its values
// at the edges added to the support of their slots.  Steps of CK columns go
// through two stages in LDS, the next ones' loads in flight in registers
// meanwhile: with the next step's alone, N = 16384 took 1.38 ms against 1.12.
// Bound by the LDS reads (a wavefront reads 4 fragments for 4 products) and
// the latency of the loads.  The workgroups of an XCD (block index mod 8) take neighbouring
// tiles of a panel, so that its L2 holds the rows that they read together.
__global__ __launch_bounds__(CBLOCK) void k_core_count(int32_t r0, int32_t N, int64_t ntiles,
                                                       const v4i *__restrict__ mat,
                                                       const int64_t *__restrict__ orp,
                                                       const int32_t *__restrict__ ocol,
                                                       uint32_t *__restrict__ osup,
                                                       unsigned long long *__restrict__ sum) {
    __shared__ v4i stage[2][STEP_WORDS];
    __shared__ uint32_t from[2][CT];
    __shared__ unsigned long long part[CBLOCK / TC_WAVE];
    const int64_t per = (ntiles + 7) / 8;
    const int64_t t = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
    if (blockIdx.x / 8 >= per || t >= ntiles) return;
    int I, J;
    core_tile(t, I, J);
    const int wv = threadIdx.x / TC_WAVE, lane = __lane_id();
    const int wr = wv >> 1, wc = wv & 1;
    // the slots of each row of the tile that lie in its columns
    {
        const int64_t u = (int64_t)r0 + I * CT + threadIdx.x % CT;
        const int side = threadIdx.x / CT;
        const int32_t key = r0 + (J + side) * CT;
        int64_t a = orp[u], b = orp[u + 1];
        while (a < b) {
            const int64_t c = (a + b) >> 1;
            if (ocol[c] < key) a = c + 1; else b = c;
        }
        from[side][threadIdx.x % CT] = (uint32_t)a;
    }
    const int64_t NR = N / 32;
    // fragment wv of the tile's rows and of its columns, for both 64-column
    // blocks of a step
    const v4i *pa = mat + ((int64_t)I * (CT / 32) + wv) * FRAG + lane;
    const v4i *pb = mat + ((int64_t)J * (CT / 32) + wv) * FRAG + lane;
    const int64_t kstep = NR * FRAG;
    v16f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    // the loads of AHEAD steps are in flight: a step's products take a tenth
    // of the time that a load takes
    v4i r[AHEAD][4];
#pragma unroll
    for (int q = 0; q < AHEAD; ++q) {
        r[q][0] = pa[0];
        r[q][1] = pa[kstep];
        r[q][2] = pb[0];
        r[q][3] = pb[kstep];
        pa += 2 * kstep;
        pb += 2 * kstep;
        __builtin_amdgcn_sched_barrier(0);  // in the order in which they are waited for
    }
    const int steps = N / CK;  // a multiple of AHEAD
    for (int s0 = 0; s0 < steps; s0 += AHEAD) {
        // the last round reads the first steps again and leaves them
        const int64_t next = s0 + AHEAD < steps ? 0 : -2 * kstep * steps;
        pa += next;
        pb += next;
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) {
            // this stage was last read two steps ago: every wavefront has
            // passed the barrier of the step between
            v4i *st = stage[q & 1];
#pragma unroll
            for (int x = 0; x < 4; ++x) st[(4 * x + wv) * FRAG + lane] = r[q][x];
            __syncthreads();
            r[q][0] = pa[0];
            r[q][1] = pa[kstep];
            r[q][2] = pb[0];
            r[q][3] = pb[kstep];
            pa += 2 * kstep;
            pb += 2 * kstep;
            __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the products
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v8i a[2], b[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const v4i x = st[(h * 4 + wr * 2 + i) * FRAG + lane];
                    const v4i y = st[(8 + h * 4 + wc * 2 + i) * FRAG + lane];
                    a[i] = v8i{x.x, x.y, x.z, x.w, 0, 0, 0, 0};
                    b[i] = v8i{y.x, y.y, y.z, y.w, 0, 0, 0, 0};
                }
                // 4-bit operands (format 4), scales 2^0
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                            a[i], b[j], acc[i][j], 4, 4, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
            }
        }
    }
    __syncthreads();
    // the tile's counts (below 2^16) in place of the stages
    uint16_t *cnt = reinterpret_cast<uint16_t *>(&stage[0][0]);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = wr * 64 + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                cnt[row * CT + wc * 64 + j * 32 + (lane & 31)] = (uint16_t)acc[i][j][e];
            }
    __syncthreads();
    // 16 lanes per row; every slot belongs to one tile
    unsigned long long total = 0;
    const int32_t c0 = r0 + J * CT;
    for (int row = threadIdx.x / 16; row < CT; row += CBLOCK / 16) {
        const uint32_t k1 = from[1][row];
        for (uint32_t k = from[0][row] + threadIdx.x % 16; k < k1; k += 16) {
            const uint32_t c = cnt[row * CT + (ocol[k] - c0)];
            if (c) osup[k] += c;
            total += c;
        }
    }
    total = tc_wave_sum(total);
    if (lane == 0) part[wv] = total;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < CBLOCK / TC_WAVE; ++w) total += part[w];
        if (total) atomicAdd(sum, total);
    }
}

// Every triangle of the core was counted at its three edges.
__global__ void k_core_found(const unsigned long long *__restrict__ sum,
                             unsigned long long *__restrict__ found) {
    *found += *sum / 3;
}

}  // namespace

// The size that saves most.  Measured on R-MAT graphs, in ps: the scan and the
// fold take 1.0 (scale 20) to 0.6 (scale 24) per wedge whose lowest end is in
// the core; the products 0.00025 N^3 (3.9 PFLOP/s at N = 16384: 1.12 ms; 1.28
// in scale 24's denser core) with about 40 us more for the launches, the
// searches and the tiles' ends, and the matrix 0.55 N^2 (144 us at 16384).  At
// scale 20 a core of 6144 takes 173 us and saves 441 of 2640 us, one of 16384
// takes 1259 us and saves 800.
int32_t tc_core_size(const tc_graph *g) {
    int32_t best = 0;
    double gain = 2e7;
    for (int j = 0; j < TC_CORE_SIZES; ++j) {
        const double N = tc_core_ranks(j);
        // the matrix fits where the transposition's sort had its buffers
        if (N > g->n || N * N / 2 > 16.0 * (double)g->m) break;
        const double x =
            (double)g->core_wedges[j] * 1.0 - (4e7 + N * N * 0.55 + N * N * N * 0.00025);
        if (x > gain) {
            gain = x;
            best = (int32_t)N;
        }
    }
    return best;
}

tc_status tc_core_fill(const tc_graph *g, int32_t N, int64_t *end, uint4 *mat, hipStream_t s) {
    const size_t lds = (size_t)FILL_ROWS * (N / 32 + FILL_ROWS) * sizeof(uint32_t);
    k_core_fill<<<(unsigned)(N / FILL_ROWS), 64 * FILL_ROWS, lds, s>>>(
        g->n - N, N, g->orp, g->ocol, g->in_ptr, g->in_pair, end, mat);
    TC_LAUNCHED();
    return TC_OK;
}

tc_status tc_core_count(const tc_graph *g, int32_t N, const uint4 *mat, unsigned long long *sum,
                        unsigned long long *found, hipStream_t s) {
    TC_TRY(tc_zero({{sum, 2}}, s));
    const int64_t T = N / CT, ntiles = T * (T + 1) / 2;
    k_core_count<<<(unsigned)((ntiles + 7) / 8 * 8), CBLOCK, 0, s>>>(
        g->n - N, N, ntiles, reinterpret_cast<const v4i *>(mat), g->orp, g->ocol, g->osup, sum);
    TC_LAUNCHED();
    k_core_found<<<1, 1, 0, s>>>(sum, found);
    TC_LAUNCHED();
    return TC_OK;
}
