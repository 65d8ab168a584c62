// Gradient statistics of Section 3 (arxiv 1802.04434): Welford's single-pass
// mean / variance over a sequence of stochastic gradients, and the density
// measure phi(v) = |v|_1^2 / (d |v|_2^2) of equation (1), with which the paper
// compares how dense gradient and noise are (Figure 1).
//
// Welford is pointwise and streams like the step kernels (20 bytes per
// coordinate: read g, mean, m2; write mean, m2).  The density is two sums over
// d elements: every term is exact in fp64, each lane accumulates its share in
// fp64, waves reduce by lane moves and blocks through LDS, each block leaves
// its pair of sums in a scratch slot and the last block to finish adds the
// slots.  Every addition happens in an order that depends on d alone, so the
// result is the same bits on every run.
#pragma once
#include "vote_apply_kernels.hpp"

namespace ss {

struct WelfordArgs {
    const void *g;
    float *mean;
    float *m2;
    float n;          // index of this gradient, 1-based, as fp32
    uint32_t n_tiles;
    size_t d;
};

// delta = g - mean; mean <- mean + delta / n; m2 <- m2 + delta * (g - mean)
__device__ __forceinline__ void welford1(float g, float n, float &mean, float &m2) {
    const float delta = g - mean;
    const float q = delta / n;
    mean = mean + q;
    const float delta2 = g - mean;
    const float p = delta * delta2;
    m2 = m2 + p;
}

// One-wave blocks of one row.  Five streams; the shapes and what is left in the memory-side cache for the next update, for sigma and
// for the densities are the host's (ss_welford_update).
template <int HOLD_KB, int STORE_MEAN, int STORE_M2, uint32_t CHUNK, typename G>
__global__ __launch_bounds__(kWave) void welford_update_kernel(const WelfordArgs a) {
    reserve_lds<HOLD_KB>(a.d == ~(size_t)0, reinterpret_cast<uint32_t *>(a.mean));
    constexpr uint32_t kGrad = kWaveCoords * sizeof(typename G::elem), kFloat = kWaveCoords * sizeof(float);
    const uint32_t lane = threadIdx.x;
    if (blockIdx.x < a.n_tiles) {
        const size_t tile = die_tile<CHUNK>(blockIdx.x, a.n_tiles);
        const Window mean_w = window(a.mean, tile * kFloat, kFloat), m2_w = window(a.m2, tile * kFloat, kFloat);
        const f32x4 gv = G::load4(window(a.g, tile * kGrad, kGrad), lane);
        f32x4 mean = ld_quad(mean_w, lane * 16);
        f32x4 m2 = ld_quad(m2_w, lane * 16);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float mean_c = mean[c], m2_c = m2[c];
            welford1(gv[c], a.n, mean_c, m2_c);
            mean[c] = mean_c;
            m2[c] = m2_c;
        }
        st_quad<STORE_MEAN>(mean_w, lane * 16, mean);
        st_quad<STORE_M2>(m2_w, lane * 16, m2);
        return;
    }
    const size_t i = a.n_tiles * (size_t)kWaveCoords + (size_t)(blockIdx.x - a.n_tiles) * kWave + lane;
    if (i < a.d) {
        float mean = a.mean[i], m2 = a.m2[i];
        welford1(G::load1(a.g, i), a.n, mean, m2);
        a.mean[i] = mean;
        a.m2[i] = m2;
    }
}

struct SigmaArgs {
    const float *m2;
    float *sigma;
    float n;
    uint32_t n_tiles;
    size_t d;
};

__device__ __forceinline__ float sigma1(float m2, float n) {
    const float var = m2 / n;
    return __builtin_sqrtf(var);
}

// R rows: one, but for vectors whose one-row grid would have 2^32 threads.  Read by address; the store policy is the host's (ss_welford_sigma).
template <int R, int STORE>
__global__ __launch_bounds__(kWave) void welford_sigma_kernel(const SigmaArgs a) {
    constexpr uint32_t kCoords = R * kWaveCoords;
    const uint32_t lane = threadIdx.x;
    const size_t tile = blockIdx.x;
    if (tile < a.n_tiles) {
        const Window to = window(a.sigma, tile * (kCoords * sizeof(float)), kCoords * sizeof(float));
        f32x4 v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = ld_stream(reinterpret_cast<const f32x4 *>(a.m2) + (tile * R + r) * kWave + lane);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            f32x4 s;
            s.x = sigma1(v[r].x, a.n);
            s.y = sigma1(v[r].y, a.n);
            s.z = sigma1(v[r].z, a.n);
            s.w = sigma1(v[r].w, a.n);
            st_quad<STORE>(to, (r * kWave + lane) * 16, s);
        }
        return;
    }
    const size_t i = a.n_tiles * (size_t)kCoords + (tile - a.n_tiles) * kWave + lane;
    if (i < a.d) a.sigma[i] = sigma1(a.m2[i], a.n);
}

// ------------------------------------------------------------- density ----
// One launch, fixed summation order.  Block b owns tiles b, b + G, b + 2G, ... of R rows of
// kDensityThreads quads (R and G = gridDim.x <= kDensityMaxBlocks, functions of d alone); the rows left over
// go to the blocks one by one.  Each lane adds its elements in that order in fp64, lanes combine
// through a tree of lane moves, waves through LDS, and the block's two sums go to slot b of a scratch array.
// The block that takes the last ticket adds the G slots in a fixed order (whichever block it is),
// writes the result and puts the ticket back to zero for the next call.  A vector of less than two
// tiles is one block's, which needs neither slots nor ticket.
//
// What does not fill a tile used to be added one coordinate a lane and turn, a chain of up to 32
// dependent loads (us): d = 1,000 3.6 -> 2.2, 10,007 5.5 -> 2.7, 40,001 5.0 -> 4.4.  Dealing all rows out
// evenly instead of whole tiles to 134 - 256 blocks costs 1 us at 4.4 M (more tickets) and gains
// nothing at 25.6 M.  After its last element a block is a chain of dependent steps; lane moves for the shuffles through LDS, one wave instead
// of eight after the waves' sums and one rounding for product and sum took 0.6 - 0.8 us off it: 272,474 5.6 -> 4.8, 4.4 M 8.0 -> 7.3, 25.6 M 19.3 -> 18.7.

// Few, large blocks: the tickets are atomics on one address and cost about 11 ns each, one after
// the other, at the very end of the launch (measured: 780 blocks of 256 threads 25 us at
// d = 25.6 M, 223 blocks of 512 threads 18 us; a plain read of the same bytes 16 us).
constexpr int kDensityMaxBlocks = 256;
constexpr int kDensityThreads = 512;

// layout of the scratch area: ticket counter, then one pair of sums per block
struct DensityScratch {
    unsigned long long ticket;           // zero between calls
    unsigned long long pad[7];
    double partial[kDensityMaxBlocks][2];
};

struct DensityArgs {
    const float *v;
    double *out;       // out[0] = |v|_1, out[1] = |v|_2^2, out[2] = phi
    DensityScratch *scratch;
    size_t d;
    size_t n_tiles;    // full tiles
    size_t n_rows;     // full rows, those of the tiles included
};

// the square of a 24-bit significand is exact, so that one rounding is what product and sum give
__device__ __forceinline__ void accumulate(float v, double &l1, double &l2sq) {
    const double a = (double)__builtin_fabsf(v);
    l1 += a;
    l2sq = __builtin_fma(a, a, l2sq);
}

// another lane's value, zero in the rows (of 16 lanes) that ROWS leaves out
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ double lane_move(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xF, false);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// sum over each eight lanes, in all of them
__device__ __forceinline__ double sum8(double s) {
    s += lane_move<0xB1 /* quad_perm [1,0,3,2] */>(s);
    s += lane_move<0x4E /* quad_perm [2,3,0,1] */>(s);
    return s + lane_move<0x141 /* row_half_mirror */>(s);
}

// sum over the wave, in lane 63
__device__ __forceinline__ double sum_wave(double s) {
    s = sum8(s);
    s += lane_move<0x140 /* row_mirror */>(s);
    s += lane_move<0x142 /* row_bcast:15 */, 0xA>(s);
    return s + lane_move<0x143 /* row_bcast:31 */, 0xC>(s);
}

__device__ __forceinline__ void density_result(const DensityArgs &a, double s1, double s2) {
    a.out[0] = s1;
    a.out[1] = s2;
    a.out[2] = s2 > 0.0 ? s1 * s1 / ((double)a.d * s2) : 0.0;
}

// the quads of N rows first, then the rows into the running sums: the longest chain of additions is
// 4 N + (batches per block), not their product
template <int N>
__device__ __forceinline__ void density_batch(const f32x4 *v, size_t row, size_t stride, double &l1, double &l2sq) {
    f32x4 q[N];
#pragma unroll
    for (int r = 0; r < N; ++r) q[r] = ld_stream(v + (row + r * stride) * kDensityThreads);
    double t1 = 0.0, t2 = 0.0;
#pragma unroll
    for (int r = 0; r < N; ++r) {
        accumulate(q[r].x, t1, t2);
        accumulate(q[r].y, t1, t2);
        accumulate(q[r].z, t1, t2);
        accumulate(q[r].w, t1, t2);
    }
    l1 += t1;
    l2sq += t2;
}

// the n <= NMAX rows that full batches leave over, as one batch of exactly that size
template <int NMAX>
__device__ __forceinline__ void density_rest(const f32x4 *v, size_t row, size_t stride, size_t n, double &l1, double &l2sq) {
    if (n == NMAX) {
        density_batch<NMAX>(v, row, stride, l1, l2sq);
    } else if constexpr (NMAX > 1) {
        density_rest<NMAX - 1>(v, row, stride, n, l1, l2sq);
    }
}

// R rows of a tile, whose loads are issued together: see density_rows in api.hip
template <int R>
__global__ __launch_bounds__(kDensityThreads) void density_kernel(const DensityArgs a) {
    constexpr int B = kDensityThreads, kWaves = B / 64;
    static_assert(kWaves == 8, "sum8 adds the waves' sums");
    __shared__ double part[2][kWaves];
    const int tid = threadIdx.x, lane = tid & 63;
    const unsigned G = gridDim.x;
    double l1 = 0.0, l2sq = 0.0;
    const f32x4 *const v = reinterpret_cast<const f32x4 *>(a.v) + tid;
    for (size_t tile = blockIdx.x; tile < a.n_tiles; tile += G) density_batch<R>(v, tile * R, 1, l1, l2sq);
    const size_t row = a.n_tiles * R + blockIdx.x;
    if (row < a.n_rows) density_rest<R - 1>(v, row, G, (a.n_rows - row + G - 1) / G, l1, l2sq);
    // what does not fill a row, by the last block: at most one quad a lane, then up to three coordinates
    if (blockIdx.x == G - 1) {
        const size_t quad = a.n_rows * B + tid;
        if (quad < a.d / kQuad) density_batch<1>(v, a.n_rows, 0, l1, l2sq);
        const size_t i = a.d / kQuad * kQuad + tid;
        if (i < a.d) accumulate(a.v[i], l1, l2sq);
    }
    l1 = sum_wave(l1);
    l2sq = sum_wave(l2sq);
    if (lane == 63) {
        part[0][tid >> 6] = l1;
        part[1][tid >> 6] = l2sq;
    }
    __syncthreads();
    if (tid >= 64) return;
    l1 = sum8(part[0][lane & (kWaves - 1)]);
    l2sq = sum8(part[1][lane & (kWaves - 1)]);
    if (G == 1) {
        if (lane == 0) density_result(a, l1, l2sq);
        return;
    }
    unsigned last = 0;
    if (lane == 0) {
        // Publish the slot, then take a ticket.  The slot is written with device-scope stores
        // (they go through to where every compute die sees them) and the wave waits until they
        // have been performed before it issues the ticket's atomic; a device-wide release fence
        // would do the same but writes back the whole L2 once per block (measured: 30 us of a
        // 50 us launch).
        __hip_atomic_store(&a.scratch->partial[blockIdx.x][0], l1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&a.scratch->partial[blockIdx.x][1], l2sq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        last = __hip_atomic_fetch_add(&a.scratch->ticket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned long long)G - 1;
    }
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    asm volatile("" ::: "memory");     // the loads below stay behind the ticket
    // every other block's slot was performed before its ticket, and this block's loads below are
    // device-scope loads issued after the last ticket came back
    constexpr int kSlots = kDensityMaxBlocks / 64;
    double s1[kSlots], s2[kSlots];
#pragma unroll
    for (int k = 0; k < kSlots; ++k) {
        const unsigned b = lane + 64 * k;
        s1[k] = b < G ? __hip_atomic_load(&a.scratch->partial[b][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
        s2[k] = b < G ? __hip_atomic_load(&a.scratch->partial[b][1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
    }
#pragma unroll
    for (int k = 1; k < kSlots; ++k) {
        s1[0] += s1[k];
        s2[0] += s2[k];
    }
    l1 = sum_wave(s1[0]);
    l2sq = sum_wave(s2[0]);
    if (lane == 63) {
        density_result(a, l1, l2sq);
        __hip_atomic_store(&a.scratch->ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace ss
