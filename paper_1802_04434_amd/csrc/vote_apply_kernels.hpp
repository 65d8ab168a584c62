// Stand-alone kernels of the three-call path: the server's majority vote over
// packed sign words and the worker's parameter update from packed bits
// (arxiv 1802.04434, Algorithm 3; Algorithm 1 when the bits are one worker's).
#pragma once
#include "step_kernels.hpp"

namespace ss {

// ---------------------------------------------------------------- vote ----
// Bit-sliced: a 32-bit word holds 32 coordinates of one worker; the M
// workers' words for the same coordinates are added "vertically" with
// carry-save adders into the binary planes of the per-coordinate count of "-"
// votes, and the count is compared with the constant threshold
// T = floor(M/2)+1 plane by plane.  32 coordinates per ALU lane-operation.

template <typename W>    // a word, or four of them
struct Sum2 { W sum, carry; };
template <typename W>
__device__ __forceinline__ Sum2<W> full_add(W a, W b, W c) {
    const W ab = a ^ b;
    return {ab ^ c, (a & b) | (ab & c)};
}
template <typename W>
__device__ __forceinline__ Sum2<W> half_add(W a, W b) { return {a ^ b, a & b}; }

// count >= T decided from the least significant plane upwards:
// ge_k = plane_k > T_k, or equal and ge_(k-1)
__device__ __forceinline__ uint32_t ge_step(uint32_t ge, uint32_t plane, int T, int k) {
    return ((T >> k) & 1) ? (plane & ge) : (plane | ge);
}

// N words of weight 2^K: reduce to one word (plane K) and N/2 carries of
// weight 2^(K+1), fold plane K into the comparison, recurse on the carries.
template <int N, int K, int T>
struct CsaLevel {
    static __device__ __forceinline__ uint32_t run(const uint32_t (&w)[N], uint32_t ge) {
        constexpr int kFull = (N - 1) / 2;
        constexpr int kNext = N / 2;
        uint32_t next[kNext > 0 ? kNext : 1];
        uint32_t acc = w[0];
#pragma unroll
        for (int j = 0; j < kFull; ++j) {
            const Sum2<uint32_t> s = full_add(acc, w[1 + 2 * j], w[2 + 2 * j]);
            acc = s.sum;
            next[j] = s.carry;
        }
        if constexpr (N % 2 == 0) {
            const Sum2<uint32_t> s = half_add(acc, w[N - 1]);
            acc = s.sum;
            next[kFull] = s.carry;
        }
        ge = ge_step(ge, acc, T, K);
        if constexpr (kNext > 0) {
            return CsaLevel<kNext, K + 1, T>::run(next, ge);
        } else {
            return ge;
        }
    }
};

// bit set where at least floor(M/2)+1 of the M words have it set
template <int M>
__device__ __forceinline__ uint32_t majority_word(const uint32_t (&w)[M]) {
    return CsaLevel<M, 0, M / 2 + 1>::run(w, 0xFFFFFFFFu);
}

template <int NPTR>
struct VoteArgs {
    const uint32_t *packed[NPTR];
    uint32_t *voted;
    int M;
    size_t d;
    size_t n_vec;   // 128-bit groups of words, padding included
};

// bits of word `wi` that lie below coordinate d
__device__ __forceinline__ uint32_t live_mask(size_t wi, size_t d) {
    const size_t lo = wi * 32;
    if (lo + 32 <= d) return 0xFFFFFFFFu;
    if (lo >= d) return 0u;
    return (1u << (unsigned)(d - lo)) - 1u;
}

// Which 128-bit group of words a lane takes.  With runs of tiles a die (CHUNK > 0) the buffers are shorter than
// 4 GiB and are addressed by 32-bit offsets.
template <uint32_t CHUNK, int BLOCK = kWave>
struct Group {
    size_t u;
    __device__ __forceinline__ explicit Group(size_t n_vec)
        : u(die_tile<CHUNK>(blockIdx.x, (uint32_t)(n_vec / BLOCK)) * (size_t)BLOCK + threadIdx.x) {}
    __device__ __forceinline__ u32x4 load(const uint32_t *base) const {
        if constexpr (CHUNK > 0)
            return ld_stream(reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(base) + (uint32_t)((uint32_t)u * 16u)));
        else return ld_stream(reinterpret_cast<const u32x4 *>(base) + u);
    }
};

template <int M, int BLOCK, int HOLD_KB, uint32_t CHUNK>
__global__ __launch_bounds__(BLOCK) void vote_kernel(const VoteArgs<M> a) {
    reserve_lds<HOLD_KB>(a.d == ~(size_t)0, a.voted);
    const Group<CHUNK, BLOCK> at(a.n_vec);
    const size_t u = at.u;
    if (u >= a.n_vec) return;
    u32x4 in[M];
#pragma unroll
    for (int w = 0; w < M; ++w) in[w] = at.load(a.packed[w]);
    if constexpr (CHUNK > 0) __builtin_amdgcn_sched_barrier(0);
    uint32_t col[M];
    u32x4 out;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int w = 0; w < M; ++w) col[w] = in[w][c];
        out[c] = majority_word<M>(col) & live_mask(4 * u + c, a.d);
    }
    st_stream(reinterpret_cast<u32x4 *>(a.voted) + u, out);
}

// Any M up to SS_MAX_WORKERS: the binary planes of the count are kept in registers and a batch of words
// is added to them at a time.
constexpr int kPlanes = 7;   // counts up to 64 < 2^7

// N words of weight 2^K into the planes from K up (what would leave the last plane is zero: M < 2^P).  Two words a full adder, so
// that eight words cost seven full adders and P - 3 half adders, two instructions each; a ripple of half adders
// from the lowest plane up for every word by itself is 8 P of them.  us, ripple / this: vote M = 24 8.8 M coordinates 7.3 / 6.7, 40 M
// 22.4 / 21.3, quorum votes M = 24 17.6 M 20.1 / 19.0, 138 M 147 / 141, M = 12 8.8 M 6.5 / 6.1; beyond, memory decides (390 M: level).
template <int K, int P, int N, typename W>
__device__ __forceinline__ void add_words(W (&plane)[P], const W (&w)[N]) {
    if constexpr (K < P) {
        W carry[(N + 1) / 2];
        W acc = plane[K];
#pragma unroll
        for (int j = 0; j < N / 2; ++j) {
            const Sum2<W> s = full_add(acc, w[2 * j], w[2 * j + 1]);
            acc = s.sum;
            carry[j] = s.carry;
        }
        if constexpr (N % 2 != 0) {
            const Sum2<W> s = half_add(acc, w[N - 1]);
            acc = s.sum;
            carry[N / 2] = s.carry;
        }
        plane[K] = acc;
        add_words<K + 1>(plane, carry);
    }
}

// NB workers' 128-bit groups loaded together (no test between the loads: all NB are in flight
// before the first is used), then added
template <int P, int NB, uint32_t CHUNK>
__device__ __forceinline__ void count_batch(const uint32_t *const *packed, const Group<CHUNK> &at, u32x4 (&plane)[P]) {
    u32x4 in[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) in[j] = at.load(packed[j]);
    __builtin_amdgcn_sched_barrier(0);
    add_words<0>(plane, in);
}

// the m <= NMAX workers that the full batches leave over, as one batch of exactly that size
template <int P, int NMAX, uint32_t CHUNK>
__device__ __forceinline__ void count_rest(const uint32_t *const *packed, int m, const Group<CHUNK> &at, u32x4 (&plane)[P]) {
    if (m == NMAX) {
        count_batch<P, NMAX>(packed, at, plane);
    } else if constexpr (NMAX > 1) {
        count_rest<P, NMAX - 1>(packed, m, at, plane);
    }
}

template <int P, int NB, uint32_t CHUNK>
__device__ __forceinline__ void count_all(const uint32_t *const *packed, int M, const Group<CHUNK> &at, u32x4 (&plane)[P]) {
#pragma unroll
    for (int k = 0; k < P; ++k) plane[k] = u32x4{0, 0, 0, 0};
    int w0 = 0;
    for (; w0 + NB <= M; w0 += NB) count_batch<P, NB>(packed + w0, at, plane);
    count_rest<P, NB - 1>(packed + w0, M - w0, at, plane);
}

template <int HOLD_KB, uint32_t CHUNK>
__global__ __launch_bounds__(kWave) void vote_kernel_any(const VoteArgs<64> a) {
    reserve_lds<HOLD_KB>(a.d == ~(size_t)0, a.voted);
    const Group<CHUNK> at(a.n_vec);
    const size_t u = at.u;
    if (u >= a.n_vec) return;
    const int T = a.M / 2 + 1;
    u32x4 plane[kPlanes];
    count_all<kPlanes, 8>(a.packed, a.M, at, plane);
    u32x4 ge = u32x4{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
#pragma unroll
    for (int k = 0; k < kPlanes; ++k) ge = ((T >> k) & 1) ? (plane[k] & ge) : (plane[k] | ge);
    ge.x &= live_mask(4 * u + 0, a.d);
    ge.y &= live_mask(4 * u + 1, a.d);
    ge.z &= live_mask(4 * u + 2, a.d);
    ge.w &= live_mask(4 * u + 3, a.d);
    st_stream(reinterpret_cast<u32x4 *>(a.voted) + u, ge);
}

// One word of every worker, added into P binary planes of the count of "-" votes; NB workers' words are
// out together.
template <int P, int NB>
__device__ __forceinline__ void count_words(const uint32_t *const *packed, int M, size_t wi, uint32_t (&plane)[P]) {
#pragma unroll
    for (int k = 0; k < P; ++k) plane[k] = 0;
    for (int w0 = 0; w0 < M; w0 += NB) {
        uint32_t word[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) word[j] = packed[w0 + j < M ? w0 + j : w0][wi];
#pragma unroll
        for (int j = 0; j < NB; ++j) word[j] = w0 + j < M ? word[j] : 0u;
        add_words<0>(plane, word);
    }
}

// The vote for a vector of a few million coordinates: one word a lane, so that there are four times the
// waves and sixteen workers' words are out at once.
__global__ __launch_bounds__(64) void vote_word_kernel(const VoteArgs<64> a) {
    const size_t wi = (size_t)blockIdx.x * 64 + threadIdx.x;
    if (wi >= 4 * a.n_vec) return;
    uint32_t plane[kPlanes];
    count_words<kPlanes, 16>(a.packed, a.M, wi, plane);
    const int T = a.M / 2 + 1;
    uint32_t ge = 0xFFFFFFFFu;
#pragma unroll
    for (int k = 0; k < kPlanes; ++k) ge = ge_step(ge, plane[k], T, k);
    a.voted[wi] = ge & live_mask(wi, a.d);
}

// --------------------------------------------------------------- apply ----

// The updates from bits, from sums and from an answer with abstentions stream x in place, 8 bytes a coordinate, and read
// little beside it.  One-wave blocks in runs of half a megabyte a die: two rows, the L2 writing back while a vector fits
// the caches (kApplySmall), one row written through beyond.  us, two rows / one row / blocks of four waves as launched before: apply 1.1 M 2.4 / 3.3 / 2.9, 4.4 M 6.7 / 7.2 / 7.2, 8.8 M 12.0 / 12.0 / 12.7, 25.6 M 32.2 / 31.5 / 33.0,
// 138 M 170 / 165 / 171, 390 M 486 / 465 / 482; sums 1.1 M 2.6 / 3.3 / 3.2, 25.6 M 35.6 / 35.1 / 35.7, 138 M 188 / 184 / 188;
// answers 1.1 M 2.7 / 3.5, 25.6 M 32.9 / 31.9 / 32.7, 138 M 172 / 166 / 170.
constexpr int kWaveCoords = kWave * kQuad;
template <bool SMALL>
struct ApplyShape {
    static constexpr int kRows = SMALL ? 2 : 1;
    static constexpr int kStore = SMALL ? kStream : kThrough;
    static constexpr uint32_t kChunk = SMALL ? 8 : 9;
    static constexpr uint32_t kCoords = kRows * kWaveCoords;
};

struct ApplyArgs {
    float *x;
    const uint32_t *bits;
    float delta;
    uint32_t n_tiles;   // blocks on the vector path
    size_t d;
};

template <bool SMALL>
__global__ __launch_bounds__(kWave) void apply_kernel(const ApplyArgs a) {
    using S = ApplyShape<SMALL>;
    const uint32_t lane = threadIdx.x;
    if (blockIdx.x < a.n_tiles) {
        const size_t tile = die_tile<S::kChunk>(blockIdx.x, a.n_tiles);
        const uint32_t *const bits = a.bits + tile * (S::kCoords / 32);
        const Window xw = window(a.x, tile * (S::kCoords * sizeof(float)), S::kCoords * sizeof(float));
        f32x4 xv[S::kRows];
        uint32_t word[S::kRows];
#pragma unroll
        for (int r = 0; r < S::kRows; ++r) {
            word[r] = bits[(r * kWave + lane) >> 3];   // 8 lanes share a word
            xv[r] = ld_quad(xw, (r * kWave + lane) * 16);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < S::kRows; ++r) {
            const uint32_t nib = word[r] >> ((lane & 7) * 4);
            f32x4 v = xv[r];
            v.x = step(v.x, a.delta, nib & 1u);
            v.y = step(v.y, a.delta, nib & 2u);
            v.z = step(v.z, a.delta, nib & 4u);
            v.w = step(v.w, a.delta, nib & 8u);
            st_quad<S::kStore>(xw, (r * kWave + lane) * 16, v);
        }
        return;
    }
    const size_t i = a.n_tiles * (size_t)S::kCoords + (size_t)(blockIdx.x - a.n_tiles) * kWave + lane;
    if (i < a.d) {
        const bool neg = (a.bits[i >> 5] >> (i & 31)) & 1u;
        a.x[i] = step(a.x[i], a.delta, neg);
    }
}

// ------------------------------------------------------- vote + apply ----
// The server's vote and the workers' update in one launch, for a step whose sign bits are in
// memory already (pack_kernel over all workers): the voted word goes from the lane that computes
// it through LDS to the lanes that own its coordinates of x, instead of through HBM and another
// launch.

template <int NPTR>
struct VoteApplyArgs {
    const uint32_t *packed[NPTR];
    uint32_t *voted;
    float *x;
    int8_t *sums;         // with count planes only, may be NULL: per-coordinate sum of signs
    float delta;
    int M;
    int sum_update;       // with count planes only: x <- x - delta * (sum of signs) instead of its sign
    size_t d;
    size_t words_total;   // words of a packed buffer including zero padding
};

// MT workers at compile time; MT == 0: a.M at run time, added into binary count planes.
// P > 0 (with MT == 0): the P planes themselves go through LDS, for the sums and the sum update.
// A block owns R rows of BLOCK quads; its first lanes vote on a word each.  Bound by HBM: 8.125 + M / 8 bytes per
// coordinate.  HOLD_KB caps the blocks per compute unit; the shapes are launch_vote_apply's.
template <int MT, int NPTR, int P, int BLOCK, int R, int HOLD_KB>
__global__ __launch_bounds__(BLOCK) void vote_apply_kernel(const VoteApplyArgs<NPTR> a) {
    reserve_lds<HOLD_KB>(a.d == ~(size_t)0, a.voted);
    constexpr int kRowCoords = BLOCK * kQuad;
    constexpr int kCoords = R * kRowCoords;
    constexpr int kWords = kCoords / 32;   // voted words of a block
    static_assert(kWords <= BLOCK, "a lane votes on one word");
    __shared__ uint32_t vote[P > 0 ? P : 1][kWords];   // the voted words, or the count planes
    const int tid = threadIdx.x;
    const size_t wi = (size_t)blockIdx.x * kWords + tid;
    const size_t base = (size_t)blockIdx.x * kCoords;
    const bool full = base + kCoords <= a.d;
    const bool votes = tid < kWords && wi < a.words_total;
    uint32_t in[MT > 0 ? MT : 1];
    if (MT > 0 && votes) {
#pragma unroll
        for (int w = 0; w < MT; ++w) in[w] = a.packed[w][wi];
    }
    const Window xw = window(a.x, base * sizeof(float), full ? kCoords * sizeof(float) : 0);
    f32x4 xv[R];
#pragma unroll
    for (int r = 0; r < R; ++r) xv[r] = ld_quad(xw, (r * BLOCK + tid) * 16);
    __builtin_amdgcn_sched_barrier(0);
    if (votes) {
        uint32_t ge;
        if constexpr (MT > 0) {
            ge = majority_word<MT>(in);
        } else {
            constexpr int N = P > 0 ? P : kPlanes;
            const int T = a.M / 2 + 1;
            uint32_t plane[N];
            count_words<N, 8>(a.packed, a.M, wi, plane);
            ge = 0xFFFFFFFFu;
#pragma unroll
            for (int k = 0; k < N; ++k) ge = ge_step(ge, plane[k], T, k);
            if constexpr (P > 0) {
#pragma unroll
                for (int k = 0; k < P; ++k) vote[k][tid] = plane[k];
            }
        }
        ge &= live_mask(wi, a.d);
        a.voted[wi] = ge;
        if constexpr (P == 0) vote[0][tid] = ge;
    }
    __syncthreads();
    if (full) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int word = r * (kRowCoords / 32) + (tid >> 3), shift = (tid & 7) * 4;
            f32x4 v = xv[r];
            if constexpr (P > 0) {
                uint32_t counts = 0;
#pragma unroll
                for (int k = 0; k < P; ++k) counts += spread_nibble((vote[k][word] >> shift) & 0xFu) << k;
                if (a.sum_update) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[c] = step_sum(v[c], a.delta, sum_at(counts, c, a.M));
                } else {
                    const uint32_t nib = vote_nibble(counts, a.M / 2 + 1);
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[c] = step(v[c], a.delta, (nib >> c) & 1u);
                }
                if (a.sums)
                    st_stream(reinterpret_cast<uint32_t *>(a.sums + base) + r * BLOCK + tid, sums_word(counts, a.M));
            } else {
                const uint32_t nib = vote[0][word] >> shift;
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = step(v[c], a.delta, (nib >> c) & 1u);
            }
            st_quad<kThrough>(xw, (r * BLOCK + tid) * 16, v);
        }
        return;
    }
    // the last block: one coordinate per lane
    for (int i = tid; base + i < a.d; i += BLOCK) {
        if constexpr (P > 0) {
            int count = 0;
#pragma unroll
            for (int k = 0; k < P; ++k) count += (int)((vote[k][i >> 5] >> (i & 31)) & 1u) << k;
            const int S = a.M - 2 * count;
            a.x[base + i] = a.sum_update ? step_sum(a.x[base + i], a.delta, S) : step(a.x[base + i], a.delta, S < 0);
            if (a.sums) a.sums[base + i] = (int8_t)S;
        } else {
            const bool neg = (vote[0][i >> 5] >> (i & 31)) & 1u;
            a.x[base + i] = step(a.x[base + i], a.delta, neg);
        }
    }
}

// ------------------------------------------------ "(good)": vote sums ----
// Section 4's first scheme sends back the sum of the workers' signs instead of
// its sign.  Bit-sliced like the vote: a lane loads 128 coordinates (four words)
// of every worker with one 128-bit load and adds them into the binary planes
// of the count of "-" votes; only at the end are the planes turned into one
// int8 per coordinate.  A lane's 128 sums are contiguous in memory, so the block
// passes them through LDS and stores them in coordinate order (a wave's store is
// 1024 contiguous bytes).

struct VoteSumArgs {
    const uint32_t *packed[64];
    int8_t *sums;
    int M;
    size_t d;
    size_t n_vec;      // 128-bit groups of packed words, padding included
};

// The planes of a word's 32 counts as bytes: byte c of out[q] is the count of coordinate 4 q + c.  The four lowest planes are
// transposed within every nibble (c[j] then holds the counts of the coordinates 4 i + j, one a nibble), nibbles are
// widened to bytes and the planes above are put in, and four words of four bytes are transposed: some 45 instructions
// for four planes where expanding each nibble of each plane by a multiplication took 200 and 32 multiplications.  With
// add_words, sums, us before / now: M = 8 8.8 M coordinates 5.4 / 4.9, 40 M 16.1 / 15.5, M = 24 4.4 M 5.7 / 5.4, M = 12 17.6 M 7.8 / 7.4.
// A single plane is expanded by multiplications (M = 1 138 M 28.6 us, transposed 28.9).
template <int P>
__device__ __forceinline__ void count_bytes(const uint32_t (&plane)[P], uint32_t (&out)[8]) {
    if constexpr (P == 1) {
#pragma unroll
        for (int q = 0; q < 8; ++q) out[q] = spread_nibble((plane[0] >> (4 * q)) & 0xFu);
        return;
    }
    const auto at = [&](int k) { return k < P ? plane[k < P ? k : 0] : 0u; };
    const auto choose = [](uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); };
    const uint32_t p0 = at(0), p1 = at(1), p2 = at(2), p3 = at(3);
    const uint32_t a01 = choose(0x55555555u, p0, p1 << 1), b01 = choose(0x55555555u, p0 >> 1, p1);
    const uint32_t a23 = choose(0x55555555u, p2, p3 << 1), b23 = choose(0x55555555u, p2 >> 1, p3);
    const uint32_t c[4] = {choose(0x33333333u, a01, a23 << 2), choose(0x33333333u, b01, b23 << 2),
                           choose(0x33333333u, a01 >> 2, a23), choose(0x33333333u, b01 >> 2, b23)};
    uint32_t even[4], odd[4];     // byte b: coordinates 8 b + j and 8 b + 4 + j
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        even[j] = c[j] & 0x0F0F0F0Fu;
        odd[j] = (c[j] >> 4) & 0x0F0F0F0Fu;
#pragma unroll
        for (int k = 4; k < P; ++k) {
            even[j] |= (plane[k] << (k - j)) & (0x01010101u << k);
            odd[j] |= (k - 4 >= j ? plane[k] << (k - 4 - j) : plane[k] >> (j + 4 - k)) & (0x01010101u << k);
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t(&v)[4] = h ? odd : even;
        const uint32_t lo01 = __builtin_amdgcn_perm(v[1], v[0], 0x05010400u), hi01 = __builtin_amdgcn_perm(v[1], v[0], 0x07030602u);
        const uint32_t lo23 = __builtin_amdgcn_perm(v[3], v[2], 0x05010400u), hi23 = __builtin_amdgcn_perm(v[3], v[2], 0x07030602u);
        out[h] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
        out[2 + h] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
        out[4 + h] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
        out[6 + h] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
    }
}

constexpr int kVoteSumLaneBytes = 128;     // a lane's 128 coordinates give 128 int8 sums
constexpr int kVoteSumLdsStride = 144;     // ... kept 144 bytes apart in LDS (spreads the banks)

// P = number of binary planes of the count of "-" votes: counts up to M < 2^P.  One-wave blocks; HOLD_KB of LDS on top of the tile,
// STORE, CHUNK and how many workers' words are loaded together (NB) by the size of the vector (launch_vote_sum)
template <int P, int HOLD_KB, int STORE, uint32_t CHUNK, int NB>
__global__ __launch_bounds__(kWave) void vote_sum_kernel(const VoteSumArgs a) {
    reserve_lds<HOLD_KB>(a.d == ~(size_t)0, reinterpret_cast<uint32_t *>(a.sums));
    __shared__ __align__(16) unsigned char tile[kWave * kVoteSumLdsStride];
    const uint32_t lane = threadIdx.x;
    Group<CHUNK> at(a.n_vec);
    const size_t base = (at.u - lane) * kVoteSumLaneBytes;
    // lanes beyond the last group (last block only) re-read the last group: their coordinates
    // lie at or beyond d and are never stored
    if (at.u >= a.n_vec) at.u = a.n_vec - 1;
    u32x4 plane[P];
    count_all<P, NB>(a.packed, a.M, at, plane);
    // planes -> one int8 sum per coordinate: the lane's 128 sums go to LDS as eight 16-byte pieces
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        uint32_t column[P], counts[8];
#pragma unroll
        for (int k = 0; k < P; ++k) column[k] = plane[k][w];
        count_bytes(column, counts);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4 piece;
#pragma unroll
            for (int e = 0; e < 4; ++e) piece[e] = sums_word(counts[4 * h + e], a.M);
            *reinterpret_cast<u32x4 *>(tile + lane * kVoteSumLdsStride + 16 * (2 * w + h)) = piece;
        }
    }
    __syncthreads();
    // ... and leave in the order of the coordinates: a store is 1024 contiguous bytes
    constexpr uint32_t kBytes = kWave * kVoteSumLaneBytes;
    if (base + kBytes <= a.d) {      // every block but the last: no test per store
        const Window to = window(a.sums, base, kBytes);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t c = j * kWave + lane;              // 16-byte piece within the block's output
            st_quad<STORE>(to, c * 16, *reinterpret_cast<const f32x4 *>(tile + (c >> 3) * kVoteSumLdsStride + 16 * (c & 7)));
        }
        return;
    }
#pragma unroll 1
    for (int j = 0; j < 8; ++j) {
        const int c = j * kWave + lane;
        const u32x4 piece = *reinterpret_cast<const u32x4 *>(tile + (c >> 3) * kVoteSumLdsStride + 16 * (c & 7));
        const size_t first = base + 16 * (size_t)c;
        if (first + 16 <= a.d) {
            st_stream(reinterpret_cast<u32x4 *>(a.sums + first), piece);
        } else if (first < a.d) {
            const uint32_t words[4] = {piece.x, piece.y, piece.z, piece.w};
            for (size_t i = first; i < a.d; ++i)
                a.sums[i] = (int8_t)(words[(i - first) >> 2] >> (8 * ((i - first) & 3)));
        }
    }
}

// The sums for a vector of a few million coordinates: one word, 32 sums, a lane.  A lane of the kernel
// above turns 128 counts into bytes, some 800 instructions one after the other, which is all the time
// a small launch takes.
template <int P>
__global__ __launch_bounds__(64) void vote_sum_word_kernel(const VoteSumArgs a) {
    const size_t wi = (size_t)blockIdx.x * 64 + threadIdx.x;
    if (wi * 32 >= a.d) return;
    uint32_t plane[P];
    count_words<P, 16>(a.packed, a.M, wi, plane);
    uint32_t out[8];
    count_bytes(plane, out);
#pragma unroll
    for (int q = 0; q < 8; ++q) out[q] = sums_word(out[q], a.M);
    if (wi * 32 + 32 <= a.d) {
        u32x4 *const to = reinterpret_cast<u32x4 *>(a.sums + wi * 32);
        to[0] = u32x4{out[0], out[1], out[2], out[3]};
        to[1] = u32x4{out[4], out[5], out[6], out[7]};
        return;
    }
#pragma unroll
    for (int i = 0; i < 32; ++i)
        if (wi * 32 + i < a.d) a.sums[wi * 32 + i] = (int8_t)(out[i >> 2] >> (8 * (i & 3)));
}

struct SumApplyArgs {
    float *x;
    const int8_t *sums;
    float delta;
    uint32_t n_tiles;
    size_t d;
};

// in the shapes of apply_kernel
template <bool SMALL>
__global__ __launch_bounds__(kWave) void sum_apply_kernel(const SumApplyArgs a) {
    using S = ApplyShape<SMALL>;
    const uint32_t lane = threadIdx.x;
    if (blockIdx.x < a.n_tiles) {
        const size_t tile = die_tile<S::kChunk>(blockIdx.x, a.n_tiles);
        const uint32_t *const sums = reinterpret_cast<const uint32_t *>(a.sums + tile * S::kCoords);
        const Window xw = window(a.x, tile * (S::kCoords * sizeof(float)), S::kCoords * sizeof(float));
        f32x4 xv[S::kRows];
        uint32_t sw[S::kRows];
#pragma unroll
        for (int r = 0; r < S::kRows; ++r) {
            sw[r] = ld_stream(sums + r * kWave + lane);
            xv[r] = ld_quad(xw, (r * kWave + lane) * 16);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < S::kRows; ++r) {
            f32x4 v = xv[r];
            v.x = step_sum(v.x, a.delta, (int)(int8_t)(sw[r] & 0xFFu));
            v.y = step_sum(v.y, a.delta, (int)(int8_t)((sw[r] >> 8) & 0xFFu));
            v.z = step_sum(v.z, a.delta, (int)(int8_t)((sw[r] >> 16) & 0xFFu));
            v.w = step_sum(v.w, a.delta, (int)(int8_t)(sw[r] >> 24));
            st_quad<S::kStore>(xw, (r * kWave + lane) * 16, v);
        }
        return;
    }
    const size_t i = a.n_tiles * (size_t)S::kCoords + (size_t)(blockIdx.x - a.n_tiles) * kWave + lane;
    if (i < a.d) a.x[i] = step_sum(a.x[i], a.delta, (int)a.sums[i]);
}

// ---------------------------------------------------------------- copy ----

struct CopyArgs {
    f32x4 *dst;
    const f32x4 *src;
    size_t n_vec;
};

// One row a wave, read by address and written through: 1.1 M floats 2.4 us against 2.6 for the L2's own write-back (and
// four-wave blocks of two rows), 60 M 71.8 / 73.2, 138 M 164.3 / 167.1, 390 M 465 / 469.
__global__ __launch_bounds__(kWave) void copy_kernel(const CopyArgs a) {
    const size_t first = blockIdx.x * (size_t)kWave;
    const size_t left = a.n_vec - first;
    const uint32_t lane = threadIdx.x;
    const Window to = window(a.dst, first * 16, left < kWave ? (uint32_t)left * 16 : kWave * 16);
    if (lane < left) st_quad<kThrough>(to, lane * 16, ld_stream(a.src + first + lane));
}

}  // namespace ss
