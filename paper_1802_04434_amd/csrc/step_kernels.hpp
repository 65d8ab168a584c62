// The streaming kernels behind ss_signum_vote_step and ss_signum_pack.
//
// step_kernel does the whole step in one pass: per worker the momentum update
// and sign of Algorithm 2 (or the plain sign of Algorithm 1), the optional
// per-worker packed bits, the majority vote and the parameter update of
// Algorithm 3, each gradient, momentum and parameter element read once and
// written once (arxiv 1802.04434).  pack_kernel does the workers' half alone,
// for one worker or for all of them in one launch.
//
// The path is bound by HBM traffic (12 bytes per worker and coordinate plus
// 8 for x, against a handful of ALU operations).  What decides how close to
// the DRAM's rate step_kernel runs, all measured on MI355X:
//
//  * The loads of a stage (BW workers x R rows, gradient and momentum) are
//    issued into registers before the first dependent operation or store: a
//    store to one worker's momentum could alias (as far as the compiler knows)
//    the next worker's loads and would otherwise serialise them.
//  * The amount of traffic in flight.  16-24 KB of outstanding loads per compute
//    unit (4-6 MB over the chip, the bandwidth-delay product) saturate HBM; more
//    only lengthens the memory system's queues and mixes more DRAM rows into
//    them, and the rate drops by 3-10 % - the more streams (workers) the worse.
//    For large d the kernel therefore takes one worker per stage (gradients alone, which are
//    short: up to eight) from one-wave blocks and the block reserves LDS that it never
//    uses (HOLD_KB), which caps the blocks that share a compute unit: 13 KB leave room
//    for eleven waves in a unit's 160 KB.  The host picks the shape (launch_step_m in api.hip).
//  * A tile costs (number of stages) x (one memory latency); the x load goes out
//    with the first stage's loads and the x store overlaps the next tile.
//    Small d is latency bound instead: there the loads of up to eight workers
//    go out together, and nothing is held back.
#pragma once
#include "common.hpp"

namespace ss {

template <int NPTR>
struct StepArgs {
    PtrTable<NPTR> p;
    float *x;
    uint32_t *voted;
    float beta, omb, delta;
    int M;               // number of workers in use (<= NPTR)
    int write_packed;    // per-worker bits wanted
    int warmup;          // Theorem 3 warm-up: signs come from g while m is still updated
    int sum_update;      // Section 4 "(good)": x <- x - delta * (sum of signs) instead of its sign
    int8_t *sums;        // may be NULL: per-coordinate sum of signs
    uint32_t n_tiles;    // blocks on the vector path
    uint32_t x_kept;     // so many of them store x with the policy STORE_X, the others with STORE
    size_t d;            // coordinates
    size_t words_total;  // words of a packed buffer including zero padding
};

// byte-wise counters: bit k of a nibble -> +1 in byte k
__device__ __forceinline__ uint32_t spread_nibble(uint32_t nib) {
    return (nib * 0x00204081u) & 0x01010101u;
}

// bits of the vote: byte k of `counts` holds how many workers are "-" at
// coordinate k of the quad; "-" wins iff that count reaches T = floor(M/2)+1
__device__ __forceinline__ uint32_t vote_nibble(uint32_t counts, int T) {
    uint32_t nib = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) nib |= (((counts >> (8 * k)) & 0xFFu) >= (uint32_t)T ? 1u : 0u) << k;
    return nib;
}

// the four sums of signs of a quad, S = M - 2 * (count of "-"), as four int8
// in one word.  Biasing every byte by 128 keeps each byte's arithmetic inside
// the byte; flipping bit 7 afterwards removes the bias modulo 256.
__device__ __forceinline__ uint32_t sums_word(uint32_t counts, int M) {
    return ((0x80808080u + (uint32_t)M * 0x01010101u) - 2u * counts) ^ 0x80808080u;
}

// Section 4 "(good)" for one coordinate: x - delta * S, product and
// difference each rounded (the file is compiled with contraction off)
__device__ __forceinline__ float step_sum(float x, float delta, int S) {
    const float t = delta * (float)S;
    return x - t;
}

__device__ __forceinline__ int sum_at(uint32_t counts, int k, int M) {
    return M - 2 * (int)((counts >> (8 * k)) & 0xFFu);
}

// One stage of the vector path: NW consecutive workers starting at w0, the R rows of a tile.
// Every load of the stage is issued before anything waits for one of them.
template <int NW, int R, int BLOCK, bool NEAR, int STORE, bool HAS_M, typename G, int NPTR>
__device__ __forceinline__ void step_stage(const StepArgs<NPTR> &a, int w0, size_t tile, uint32_t tid, uint32_t (&counts)[R]) {
    constexpr uint32_t kCoords = R * BLOCK * kQuad;
    constexpr uint32_t kGrad = kCoords * sizeof(typename G::elem), kFloat = kCoords * sizeof(float);
    f32x4 gv[R][NW], mv[R][NW];
#pragma unroll
    for (int j = 0; j < NW; ++j) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            gv[r][j] = G::template load_tile<NEAR>(a.p.g[w0 + j], tile, kGrad, r * BLOCK + tid);
            if (HAS_M) mv[r][j] = ld_tile<NEAR>(a.p.m[w0 + j], tile, kFloat, (r * BLOCK + tid) * 16);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NW; ++j) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            f32x4 v = gv[r][j];
            if (HAS_M) {
                f32x4 m0 = mv[r][j];
                v.x = momentum(a.beta, a.omb, m0.x, v.x);
                v.y = momentum(a.beta, a.omb, m0.y, v.y);
                v.z = momentum(a.beta, a.omb, m0.z, v.z);
                v.w = momentum(a.beta, a.omb, m0.w, v.w);
                st_tile<NEAR, STORE>(a.p.m[w0 + j], tile, kFloat, (r * BLOCK + tid) * 16, v);
            }
            // Algorithm 2 votes with sign(m); a warm-up iteration with sign(g)
            const uint32_t nib = neg_nibble((HAS_M && a.warmup) ? gv[r][j] : v);
            counts[r] += spread_nibble(nib);
            if (a.write_packed) {
                const uint32_t word = combine8(nib, tid & 63);
                if ((tid & 7) == 0) a.p.packed[w0 + j][tile * (kCoords / 32) + ((r * BLOCK + tid) >> 3)] = word;
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

// the n <= NMAX workers that the full stages leave over, as one stage of exactly that size
template <int NMAX, int R, int BLOCK, bool NEAR, int STORE, bool HAS_M, typename G, int NPTR>
__device__ __forceinline__ void step_rest(const StepArgs<NPTR> &a, int w0, int n, size_t tile, uint32_t tid, uint32_t (&counts)[R]) {
    if (n == NMAX) {
        step_stage<NMAX, R, BLOCK, NEAR, STORE, HAS_M, G>(a, w0, tile, tid, counts);
    } else if constexpr (NMAX > 1) {
        step_rest<NMAX - 1, R, BLOCK, NEAR, STORE, HAS_M, G>(a, w0, n, tile, tid, counts);
    }
}

// Scalar path for what does not fill a tile: one coordinate per lane, so
// the 64-bit wave ballot is two packed words in order.  It also writes
// the zero padding words.
template <bool HAS_M, typename G, int NPTR>
__device__ __forceinline__ void step_tail(const StepArgs<NPTR> &a, int M, size_t i, int lane) {
    const bool in = i < a.d;
    const size_t word = i >> 5;   // for lanes 0 and 32: the word this half-wave fills
    const bool writes_word = (lane & 31) == 0 && word < a.words_total;
    const int T = M / 2 + 1;
    int count = 0;
    for (int w = 0; w < M; ++w) {
        float v = 0.0f;
        if (in) {
            const float gi = G::load1(a.p.g[w], i);
            v = gi;
            if (HAS_M) {
                v = momentum(a.beta, a.omb, a.p.m[w][i], gi);
                a.p.m[w][i] = v;
                if (a.warmup) v = gi;
            }
        }
        const bool neg = in && v < 0.0f;
        count += neg ? 1 : 0;
        if (a.write_packed) {
            const uint64_t mask = __builtin_amdgcn_ballot_w64(neg);
            if (writes_word) a.p.packed[w][word] = (uint32_t)(lane == 0 ? mask : mask >> 32);
        }
    }
    const bool vneg = in && count >= T;
    if (in) {
        a.x[i] = a.sum_update ? step_sum(a.x[i], a.delta, M - 2 * count) : step(a.x[i], a.delta, vneg);
        if (a.sums) a.sums[i] = (int8_t)(M - 2 * count);
    }
    const uint64_t mask = __builtin_amdgcn_ballot_w64(vneg);
    if (writes_word) a.voted[word] = (uint32_t)(lane == 0 ? mask : mask >> 32);
}

// MT  > 0: number of workers known at compile time (M == MT)
// MT == 0: a.M workers, looped at run time
// BLOCK  : threads per block (a row is BLOCK * 4 coordinates)
// BW     : workers per stage (whose loads are issued together); what M leaves
//          over after the full stages is one smaller stage
// R      : rows per block
// HOLD_KB: kilobytes of LDS the block reserves and never uses, which caps how
//          many blocks share a compute unit (0: no cap)
// NEAR   : buffers of less than 4 GiB, addressed without arithmetic (ld_tile);  STORE, STORE_X: policies of the stores of m
//          and of x;  CHUNK: log2 of the tiles that a die takes at a time (die_tile)
template <int MT, int NPTR, int BLOCK, int BW, int R, int HOLD_KB, bool NEAR, int STORE, int STORE_X, uint32_t CHUNK, bool HAS_M, typename G>
__global__ __launch_bounds__(BLOCK) void step_kernel(const StepArgs<NPTR> a) {
    const uint32_t tid = threadIdx.x;
    const int lane = tid & 63;
    const int M = MT > 0 ? MT : a.M;
    const int T = M / 2 + 1;
    constexpr uint32_t kCoords = R * BLOCK * kQuad;
    reserve_lds<HOLD_KB>(a.d == ~(size_t)0 /* the host rejects such a d */, a.p.packed[0]);

    if (blockIdx.x < a.n_tiles) {
        const size_t tile = die_tile<CHUNK>(blockIdx.x, a.n_tiles);
        uint32_t counts[R];
        f32x4 xv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            counts[r] = 0;
            xv[r] = ld_tile<NEAR>(a.x, tile, kCoords * sizeof(float), (r * BLOCK + tid) * 16);
        }
        int w0 = 0;
        for (; w0 + BW <= M; w0 += BW) step_stage<BW, R, BLOCK, NEAR, STORE, HAS_M, G>(a, w0, tile, tid, counts);
        if constexpr (MT > 0) {
            if constexpr (MT % BW != 0) step_stage<MT % BW, R, BLOCK, NEAR, STORE, HAS_M, G>(a, w0, tile, tid, counts);
        } else if constexpr (BW > 1) {
            step_rest<BW - 1, R, BLOCK, NEAR, STORE, HAS_M, G>(a, w0, M - w0, tile, tid, counts);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t nib = vote_nibble(counts[r], T);
            f32x4 v = xv[r];
            if (a.sum_update) {
                v.x = step_sum(v.x, a.delta, sum_at(counts[r], 0, M));
                v.y = step_sum(v.y, a.delta, sum_at(counts[r], 1, M));
                v.z = step_sum(v.z, a.delta, sum_at(counts[r], 2, M));
                v.w = step_sum(v.w, a.delta, sum_at(counts[r], 3, M));
            } else {
                v.x = step(v.x, a.delta, nib & 1u);
                v.y = step(v.y, a.delta, nib & 2u);
                v.z = step(v.z, a.delta, nib & 4u);
                v.w = step(v.w, a.delta, nib & 8u);
            }
            if (STORE == STORE_X || tile < a.x_kept) st_tile<NEAR, STORE_X>(a.x, tile, kCoords * sizeof(float), (r * BLOCK + tid) * 16, v);
            else st_tile<NEAR, STORE>(a.x, tile, kCoords * sizeof(float), (r * BLOCK + tid) * 16, v);
            if (a.sums) reinterpret_cast<uint32_t *>(a.sums)[tile * (kCoords / 4) + r * BLOCK + tid] = sums_word(counts[r], M);
            const uint32_t word = combine8(nib, lane);
            if ((lane & 7) == 0) a.voted[tile * (kCoords / 32) + ((r * BLOCK + tid) >> 3)] = word;
        }
        return;
    }

    step_tail<HAS_M, G>(a, M, a.n_tiles * (size_t)kCoords + (size_t)(blockIdx.x - a.n_tiles) * BLOCK + tid, lane);
}

// The whole step for bf16 gradients without momentum.  The quad geometry would load 64 bits of gradient a
// lane; here a lane loads 128 bits, an octet of coordinates, and counts its votes in two words of byte
// counters.  x stays in quads - two per lane, whole kilobytes per wave - and what a lane needs of
// its quads' votes comes from the octets' lanes by two lane reads at the end.  Per-worker bits are not
// written here: a step of this size that wants them runs as two launches.
template <int NW, int NPTR>
__device__ __forceinline__ void octet_stage(const StepArgs<NPTR> &a, int w0, size_t o, uint32_t &lo, uint32_t &hi) {
    u32x4 gv[NW];    // eight bf16, the lower coordinate in the lower half of a word
#pragma unroll
    for (int j = 0; j < NW; ++j) gv[j] = ld_stream(reinterpret_cast<const u32x4 *>(a.p.g[w0 + j]) + o);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        const uint32_t byte = neg_byte_bf16(gv[j]);
        lo += spread_nibble(byte & 0xFu);
        hi += spread_nibble(byte >> 4);
    }
    __builtin_amdgcn_sched_barrier(0);
}

template <int NMAX, int NPTR>
__device__ __forceinline__ void octet_rest(const StepArgs<NPTR> &a, int w0, int n, size_t o, uint32_t &lo, uint32_t &hi) {
    if (n == NMAX) {
        octet_stage<NMAX>(a, w0, o, lo, hi);
    } else if constexpr (NMAX > 1) {
        octet_rest<NMAX - 1>(a, w0, n, o, lo, hi);
    }
}

// BW, HOLD_KB as for step_kernel; a tile is one row of BLOCK octets.  Up to eight workers the first x_kept tiles leave x in the memory-side
// cache: us at 25.6 M coordinates, M = 8, none of x / 75 MB of it, the same state 96.8 / 93.3, three in turn 97.2 / 92.9, twelve 98.2 / 101.1 (see kKeepX)
template <int MT, int NPTR, int BLOCK, int BW, int HOLD_KB, int STORE, int STORE_X>
__global__ __launch_bounds__(BLOCK) void step_bf16_kernel(const StepArgs<NPTR> a) {
    reserve_lds<HOLD_KB>(a.d == ~(size_t)0, a.p.packed[0]);
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63;
    const int M = MT > 0 ? MT : a.M;
    const int T = M / 2 + 1;
    constexpr uint32_t kCoords = BLOCK * 2 * kQuad;
    if (blockIdx.x < a.n_tiles) {
        const size_t o = blockIdx.x * (size_t)BLOCK + tid;
        const Window xw = window(a.x, blockIdx.x * (size_t)(kCoords * sizeof(float)), kCoords * sizeof(float));
        const uint32_t xo = (2 * (tid - lane) + lane) * 16;    // this lane's quads lie here and a kilobyte further
        uint32_t lo = 0, hi = 0;
        f32x4 xv[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) xv[h] = ld_quad(xw, xo + 1024 * h);
        int w0 = 0;
        for (; w0 + BW <= M; w0 += BW) octet_stage<BW>(a, w0, o, lo, hi);
        if constexpr (MT > 0) {
            if constexpr (MT % BW != 0) octet_stage<MT % BW>(a, w0, o, lo, hi);
        } else {
            octet_rest<BW - 1>(a, w0, M - w0, o, lo, hi);
        }
        const uint32_t byte = vote_nibble(lo, T) | (vote_nibble(hi, T) << 4);
        const uint32_t word = combine4(byte, lane);
        if ((lane & 3) == 0) a.voted[o >> 2] = word;
        if (a.sums) reinterpret_cast<uint64_t *>(a.sums)[o] = sums_word(lo, M) | ((uint64_t)sums_word(hi, M) << 32);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // quad `lane` of half h lies in the octet of lane 32 h + lane / 2
            const int from = 32 * h + (lane >> 1);
            f32x4 v = xv[h];
            if (a.sum_update) {
                const uint32_t l = (uint32_t)__shfl((int)lo, from, 64), u = (uint32_t)__shfl((int)hi, from, 64);
                const uint32_t counts = (lane & 1) ? u : l;
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = step_sum(v[c], a.delta, sum_at(counts, c, M));
            } else {
                const uint32_t nib = (uint32_t)__shfl((int)byte, from, 64) >> ((lane & 1) * 4);
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = step(v[c], a.delta, (nib >> c) & 1u);
            }
            if (STORE == STORE_X || blockIdx.x < a.x_kept) st_quad<STORE_X>(xw, xo + 1024 * h, v);
            else st_quad<STORE>(xw, xo + 1024 * h, v);
        }
        return;
    }
    step_tail<false, Bf16Grad>(a, M, a.n_tiles * (size_t)kCoords + (size_t)(blockIdx.x - a.n_tiles) * BLOCK + tid, lane);
}

// ---------------------------------------------------------------- pack ----

struct PackWorker {
    const void *g;
    float *m;            // NULL without momentum
    uint32_t *packed;
};

template <int NPTR>
struct PackArgs {
    PackWorker w[NPTR];  // blockIdx.y selects the worker
    float beta, omb;
    int warmup;          // Theorem 3 warm-up: signs come from g while m is still updated
    uint32_t n_tiles;    // blocks on the vector path, R rows of BLOCK * 4 coordinates each
    size_t d;
    size_t words_total;  // words of a packed buffer including zero padding
};

// What does not fill a tile, and the zero padding: one coordinate per lane, the wave ballot is two
// packed words in order.
template <bool HAS_M, typename G, int NPTR>
__device__ __forceinline__ void pack_tail(const PackArgs<NPTR> &a, const PackWorker &w, size_t i, int lane) {
    const bool in = i < a.d;
    float v = 0.0f;
    if (in) {
        const float gi = G::load1(w.g, i);
        v = gi;
        if (HAS_M) {
            v = momentum(a.beta, a.omb, w.m[i], gi);
            w.m[i] = v;
            if (a.warmup) v = gi;
        }
    }
    const uint64_t mask = __builtin_amdgcn_ballot_w64(in && v < 0.0f);
    const size_t word = i >> 5;
    if ((lane & 31) == 0 && word < a.words_total) w.packed[word] = (uint32_t)(lane == 0 ? mask : mask >> 32);
}

// Momentum update, sign and packed bits of Algorithm 2 for NPTR >= gridDim.y workers (m == NULL:
// Algorithm 1's sign of g).  Bound by HBM: 12.125 bytes per worker and coordinate with fp32
// gradients.  The grid is worker-major - all of a worker's tiles, then the next worker's - so that
// only three buffers are open chip-wide at a time, and a launch over all workers has one tail
// where M launches have M.
//
// With momentum a block is ONE wave with one row: the dispatcher refills a finished wave's slot at
// once, where a block of four holds its slots until its slowest wave is done (d = 138 M, M = 16, us: 3,938 against 4,106
// for four waves of one row and 4,435 for four rows; two rows a wave, neighbouring or eight apart: 4-8 % slower).
// HOLD_KB, STORE and CHUNK are chosen by the host's launch_pack_momentum: d = 25.6 M, M = 7 315 us (6,890 GB/s) where
// 64-bit addresses, the L2's own write-back and tiles in order gave 327, d = 138 M, M = 4 968 (6,935 GB/s) / 1,001,
// d = 400 M, M = 2 bf16 1,192 / 1,214.
template <int NPTR, int BLOCK, int R, int HOLD_KB, int STORE, uint32_t CHUNK, bool HAS_M, typename G>
__global__ __launch_bounds__(BLOCK) void pack_kernel(const PackArgs<NPTR> a) {
    reserve_lds<HOLD_KB>(a.d == ~(size_t)0 /* the host rejects such a d */, a.w[0].packed);
    const PackWorker w = a.w[NPTR == 1 ? 0 : blockIdx.y];
    constexpr uint32_t kCoords = R * BLOCK * kQuad;
    const uint32_t tid = threadIdx.x;
    const int lane = tid & 63;
    if (blockIdx.x < a.n_tiles) {
        const size_t tile = die_tile<CHUNK>(blockIdx.x, a.n_tiles);
        uint32_t *const out = w.packed + tile * (kCoords / 32);
        if constexpr (HAS_M) {
            const Window gw = window(w.g, tile * (kCoords * sizeof(typename G::elem)), kCoords * sizeof(typename G::elem));
            const Window mw = window(w.m, tile * (kCoords * sizeof(float)), kCoords * sizeof(float));
            f32x4 gv[R], mv[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                gv[r] = G::load4(gw, r * BLOCK + tid);
                mv[r] = ld_quad(mw, (r * BLOCK + tid) * 16);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                f32x4 v;
                v.x = momentum(a.beta, a.omb, mv[r].x, gv[r].x);
                v.y = momentum(a.beta, a.omb, mv[r].y, gv[r].y);
                v.z = momentum(a.beta, a.omb, mv[r].z, gv[r].z);
                v.w = momentum(a.beta, a.omb, mv[r].w, gv[r].w);
                st_quad<STORE>(mw, (r * BLOCK + tid) * 16, v);
                const uint32_t word = combine8(neg_nibble(a.warmup ? gv[r] : v), lane);
                if ((lane & 7) == 0) out[(r * BLOCK + tid) >> 3] = word;
            }
        } else {
            f32x4 gv[R];
#pragma unroll
            for (int r = 0; r < R; ++r) gv[r] = G::load4(w.g, (tile * R + r) * BLOCK + tid);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t word = combine8(neg_nibble(gv[r]), lane);
                if ((lane & 7) == 0) out[(r * BLOCK + tid) >> 3] = word;
            }
        }
        return;
    }
    pack_tail<HAS_M, G>(a, w, a.n_tiles * (size_t)kCoords + (size_t)(blockIdx.x - a.n_tiles) * BLOCK + tid, lane);
}

// pack_kernel for bf16 gradients without momentum: a lane loads 128 bits - eight coordinates, one
// byte of signs - and four lanes share a word.  The quad geometry above halves the gradient's
// loads to 64 bits and doubles their number: d = 25.6 M, M = 8 68 us (6,390 GB/s) against 78 with
// four rows of 256 threads and quads, d = 138 M, M = 16 720 us against 833, one worker at 25.6 M
// 9.8 against 10.8.
template <int NPTR, int BLOCK, int R, uint32_t CHUNK>
__global__ __launch_bounds__(BLOCK) void pack_bf16_kernel(const PackArgs<NPTR> a) {
    const PackWorker w = a.w[NPTR == 1 ? 0 : blockIdx.y];
    constexpr uint32_t kCoords = R * BLOCK * 2 * kQuad;
    const uint32_t tid = threadIdx.x;
    const int lane = tid & 63;
    if (blockIdx.x < a.n_tiles) {
        const size_t tile = die_tile<CHUNK>(blockIdx.x, a.n_tiles);
        u32x4 gv[R];    // eight bf16, the lower coordinate in the lower half of a word
#pragma unroll
        for (int r = 0; r < R; ++r) gv[r] = ld_stream(reinterpret_cast<const u32x4 *>(w.g) + (tile * R + r) * BLOCK + tid);
        __builtin_amdgcn_sched_barrier(0);
        uint32_t *const out = w.packed + tile * (kCoords / 32);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t word = combine4(neg_byte_bf16(gv[r]), lane);
            if ((lane & 3) == 0) out[(r * BLOCK + tid) >> 2] = word;
        }
        return;
    }
    pack_tail<false, Bf16Grad>(a, w, a.n_tiles * (size_t)kCoords + (size_t)(blockIdx.x - a.n_tiles) * BLOCK + tid, lane);
}

}  // namespace ss
