// Gradient statistics of Section 3 (arxiv 1802.04434): Welford's single-pass
// mean / variance over a sequence of stochastic gradients, and the density
// measure phi(v) = |v|_1^2 / (d |v|_2^2) of equation (1), with which the paper
// compares how dense gradient and noise are (Figure 1).
//
// Welford is pointwise and streams like the step kernels (20 bytes per
// coordinate: read g, mean, m2; write mean, m2).  The density is two sums over
// d elements: every term is exact in fp64, each lane accumulates its share in
// fp64, waves and blocks reduce through shuffles and LDS, each block leaves
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

// One-wave blocks of one row.  Five streams; the shapes are the host's (ss_welford_update), us, now / before (addresses a
// lane, the L2's own write-back): 25.6 M coordinates 77.6 / 80.0, 138 M 411 / 427, 390 M 1,148 / 1,197, bf16 138 M 366 / 384.
template <int HOLD_KB, int STORE, uint32_t CHUNK, typename G>
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
        st_quad<STORE>(mean_w, lane * 16, mean);
        st_quad<STORE>(m2_w, lane * 16, m2);
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

// R rows: one, but for vectors whose one-row grid would have 2^32 threads.  Read by address; written through (138 M 163.7 us
// against 167.7, 390 M 458 / 466) unless the vector is small enough for a cache to hold what the next kernel reads: update,
// sigma and the two densities at 1.1 M 19.7 / 18.6, at 4.4 M 39.1 / 38.0, at 17.6 M 107.2 / 108.6.
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
// One launch, fixed summation order.  Block b owns tiles b, b + G, b + 2G, ... of kDensityRows rows of
// kDensityThreads quads (G = gridDim.x <= kDensityMaxBlocks, a function of d alone); the rows left over
// go to the blocks one by one.  Each lane adds its elements in that order in fp64, lanes combine
// through a shuffle tree, waves through LDS, and the block's two sums go to slot b of a scratch array.
// The block that takes the last ticket adds the G slots in a fixed order (whichever block it is),
// writes the result and puts the ticket back to zero for the next call.  A vector of less than two
// tiles is one block's, which needs neither slots nor ticket.
//
// What does not fill a tile used to be added one coordinate a lane and turn, a chain of up to 32
// dependent loads (us): d = 1,000 3.6 -> 2.2, 10,007 5.5 -> 2.7, 40,001 5.0 -> 4.4.  Dealing all rows out
// evenly instead of whole tiles to 134 - 256 blocks costs 1 us at 4.4 M (more tickets) and gains
// nothing at 25.6 M.

// Few, large blocks: the tickets are atomics on one address and cost about 11 ns each, one after
// the other, at the very end of the launch (measured: 780 blocks of 256 threads 25 us at
// d = 25.6 M, 223 blocks of 512 threads 18 us; a plain read of the same bytes 16 us).
constexpr int kDensityMaxBlocks = 256;
constexpr int kDensityThreads = 512;
constexpr int kDensityRows = 8;          // rows of a tile, whose loads are issued together

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

__device__ __forceinline__ void accumulate(float v, double &l1, double &l2sq) {
    const double a = (double)__builtin_fabsf(v);
    l1 += a;
    l2sq += a * a;     // exact product of two 24-bit significands
}

// sum over the block of each lane's (s1, s2), in a fixed order; valid in thread 0
__device__ __forceinline__ void block_sum(double &s1, double &s2, double (*part)[kDensityThreads / 64]) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        s1 += __shfl_down(s1, off, 64);
        s2 += __shfl_down(s2, off, 64);
    }
    const int tid = threadIdx.x;
    if ((tid & 63) == 0) {
        part[0][tid >> 6] = s1;
        part[1][tid >> 6] = s2;
    }
    __syncthreads();
    if (tid == 0) {
        s1 = part[0][0];
        s2 = part[1][0];
#pragma unroll
        for (int w = 1; w < kDensityThreads / 64; ++w) {
            s1 += part[0][w];
            s2 += part[1][w];
        }
    }
    __syncthreads();
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

__global__ __launch_bounds__(kDensityThreads) void density_kernel(const DensityArgs a) {
    constexpr int R = kDensityRows;
    constexpr int B = kDensityThreads;
    __shared__ double part[2][B / 64];
    __shared__ int is_last;
    const int tid = threadIdx.x;
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
    block_sum(l1, l2sq, part);
    if (G == 1) {
        if (tid == 0) density_result(a, l1, l2sq);
        return;
    }
    if (tid == 0) {
        // Publish the slot, then take a ticket.  The slot is written with device-scope stores
        // (they go through to where every compute die sees them) and the wave waits until they
        // have been performed before it issues the ticket's atomic; a device-wide release fence
        // would do the same but writes back the whole L2 once per block (measured: 30 us of a
        // 50 us launch).
        __hip_atomic_store(&a.scratch->partial[blockIdx.x][0], l1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&a.scratch->partial[blockIdx.x][1], l2sq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        is_last = __hip_atomic_fetch_add(&a.scratch->ticket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                  (unsigned long long)G - 1;
    }
    __syncthreads();
    if (!is_last) return;
    // every other block's slot was performed before its ticket, and this block's loads below are
    // device-scope loads issued after the last ticket came back
    double s1 = 0.0, s2 = 0.0;
    for (unsigned b = tid; b < G; b += B) {
        s1 += __hip_atomic_load(&a.scratch->partial[b][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s2 += __hip_atomic_load(&a.scratch->partial[b][1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    block_sum(s1, s2, part);
    if (tid == 0) {
        density_result(a, s1, s2);
        __hip_atomic_store(&a.scratch->ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace ss
