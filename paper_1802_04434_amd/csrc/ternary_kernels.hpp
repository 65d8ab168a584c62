// "Majority vote with abstention", the ternary extension sketched in the
// Discussion (Section 6) of arxiv 1802.04434: a worker that is unsure about a
// coordinate sends 0 instead of a sign, and the server sends 0 back unless a
// quorum agrees.
//
// The paper gives no criterion, so this is a READING, stated in the header of
// the library: a worker abstains where |v| < tau (v = its momentum, or its
// gradient when there is none); the server sums the votes S = #plus - #minus
// and answers sign(S) if |S| >= Q, otherwise 0; x moves by -delta * answer.
// A ternary vector travels as two bit planes in the usual packed layout,
// "negative" and "zero" (never both set).
//
// The kernels mirror the binary ones: a streaming kernel for the worker's pack
// and for the fused step (same lane geometry and stages, optional cap on resident
// blocks through an LDS reservation), a small server kernel and an apply kernel.
#pragma once
#include "step_kernels.hpp"
#include "vote_apply_kernels.hpp"

namespace ss {

struct TernaryStepArgs {
    const void *g[64];
    float *m[64];          // all NULL without momentum
    uint32_t *neg_out;     // pack only: the planes of worker 0; the next worker's lie plane_stride words
    uint32_t *zero_out;    // further (blockIdx.y selects the worker)
    size_t plane_stride;
    float *x;              // fused only
    uint32_t *voted_neg;
    uint32_t *voted_zero;
    float beta, omb, delta, tau;
    int M;
    int quorum;
    uint32_t n_tiles;
    size_t d;
    size_t words_total;
};

// answer for one coordinate from its counts: bit 0 = negative, bit 1 = zero
__device__ __forceinline__ uint32_t quorum_answer(int n_neg, int n_zero, int M, int Q) {
    const int S = M - n_zero - 2 * n_neg;
    return S <= -Q ? 1u : (S < Q ? 2u : 0u);
}

__device__ __forceinline__ float step_ternary(float x, float delta, uint32_t answer) {
    return (answer & 2u) ? x : ((answer & 1u) ? x + delta : x - delta);
}

// One stage of the vector path: NW consecutive workers starting at w0, the R rows of a wave's tile (as step_stage of the
// binary kernel)
template <int NW, int R, bool NEAR, int STORE, bool HAS_M, bool VOTE, typename G>
__device__ __forceinline__ void ternary_stage(const TernaryStepArgs &a, int w0, size_t tile, uint32_t lane,
                                              uint32_t (&n_neg)[R], uint32_t (&n_zero)[R]) {
    constexpr uint32_t kCoords = R * kWave * kQuad;
    constexpr uint32_t kGrad = kCoords * sizeof(typename G::elem), kFloat = kCoords * sizeof(float);
    f32x4 gv[R][NW], mv[R][NW];
#pragma unroll
    for (int j = 0; j < NW; ++j) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            // what is only read has 64-bit addresses
            if (HAS_M || VOTE) gv[r][j] = G::template load_tile<NEAR>(a.g[w0 + j], tile, kGrad, r * kWave + lane);
            else gv[r][j] = G::load4(a.g[w0 + j], (tile * R + r) * kWave + lane);
            if (HAS_M) mv[r][j] = ld_tile<NEAR>(a.m[w0 + j], tile, kFloat, (r * kWave + lane) * 16);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NW; ++j) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            f32x4 v = gv[r][j];
            if (HAS_M) {
                const f32x4 m0 = mv[r][j];
                v.x = momentum(a.beta, a.omb, m0.x, v.x);
                v.y = momentum(a.beta, a.omb, m0.y, v.y);
                v.z = momentum(a.beta, a.omb, m0.z, v.z);
                v.w = momentum(a.beta, a.omb, m0.w, v.w);
                st_tile<NEAR, STORE>(a.m[w0 + j], tile, kFloat, (r * kWave + lane) * 16, v);
            }
            uint32_t zero_nib = 0, neg_nib = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const bool abstain = __builtin_fabsf(v[c]) < a.tau;
                zero_nib |= (abstain ? 1u : 0u) << c;
                neg_nib |= ((!abstain && v[c] < 0.0f) ? 1u : 0u) << c;
            }
            if (VOTE) {
                n_neg[r] += spread_nibble(neg_nib);
                n_zero[r] += spread_nibble(zero_nib);
            } else {
                const uint32_t nw = combine8(neg_nib, lane);
                const uint32_t zw = combine8(zero_nib, lane);
                if ((lane & 7) == 0) {
                    const size_t word = w0 * a.plane_stride + tile * (kCoords / 32) + ((r * kWave + lane) >> 3);
                    a.neg_out[word] = nw;
                    a.zero_out[word] = zw;
                }
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

// the n <= NMAX workers that the full stages leave over, as one stage of exactly that size
template <int NMAX, int R, bool NEAR, int STORE, bool HAS_M, bool VOTE, typename G>
__device__ __forceinline__ void ternary_rest(const TernaryStepArgs &a, int w0, int n, size_t tile, uint32_t lane,
                                             uint32_t (&n_neg)[R], uint32_t (&n_zero)[R]) {
    if (n == NMAX) {
        ternary_stage<NMAX, R, NEAR, STORE, HAS_M, VOTE, G>(a, w0, tile, lane, n_neg, n_zero);
    } else if constexpr (NMAX > 1) {
        ternary_rest<NMAX - 1, R, NEAR, STORE, HAS_M, VOTE, G>(a, w0, n, tile, lane, n_neg, n_zero);
    }
}

// One-wave blocks.  VOTE: the whole step; otherwise worker blockIdx.y's pack.  BW workers per stage (what M leaves over
// is one smaller stage), R rows per block, HOLD_KB of LDS reserved to cap the blocks per compute unit; NEAR, STORE and
// CHUNK as step_kernel's
template <int BW, int R, int HOLD_KB, bool NEAR, int STORE, uint32_t CHUNK, bool HAS_M, bool VOTE, typename G>
__global__ __launch_bounds__(kWave) void ternary_step_kernel(const TernaryStepArgs a) {
    const uint32_t lane = threadIdx.x;
    const int M = a.M;
    constexpr uint32_t kCoords = R * kWave * kQuad;
    reserve_lds<HOLD_KB>(a.d == ~(size_t)0 /* the host rejects such a d */, VOTE ? a.voted_neg : a.neg_out);

    if (blockIdx.x < a.n_tiles) {
        const size_t tile = die_tile<CHUNK>(blockIdx.x, a.n_tiles);
        uint32_t n_neg[R], n_zero[R];
        f32x4 xv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            n_neg[r] = 0;
            n_zero[r] = 0;
            if (VOTE) xv[r] = ld_tile<NEAR>(a.x, tile, kCoords * sizeof(float), (r * kWave + lane) * 16);
        }
        if constexpr (VOTE) {
            int w0 = 0;
            for (; w0 + BW <= M; w0 += BW) ternary_stage<BW, R, NEAR, STORE, HAS_M, true, G>(a, w0, tile, lane, n_neg, n_zero);
            if constexpr (BW > 1) ternary_rest<BW - 1, R, NEAR, STORE, HAS_M, true, G>(a, w0, M - w0, tile, lane, n_neg, n_zero);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                uint32_t neg_nib = 0, zero_nib = 0;
                f32x4 v = xv[r];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint32_t ans = quorum_answer((int)((n_neg[r] >> (8 * c)) & 0xFFu),
                                                       (int)((n_zero[r] >> (8 * c)) & 0xFFu), M, a.quorum);
                    neg_nib |= (ans & 1u) << c;
                    zero_nib |= ((ans >> 1) & 1u) << c;
                    v[c] = step_ternary(v[c], a.delta, ans);
                }
                st_tile<NEAR, STORE>(a.x, tile, kCoords * sizeof(float), (r * kWave + lane) * 16, v);
                const uint32_t nw = combine8(neg_nib, lane);
                const uint32_t zw = combine8(zero_nib, lane);
                if ((lane & 7) == 0) {
                    const size_t word = tile * (kCoords / 32) + ((r * kWave + lane) >> 3);
                    a.voted_neg[word] = nw;
                    a.voted_zero[word] = zw;
                }
            }
        } else {
            ternary_stage<1, R, NEAR, STORE, HAS_M, false, G>(a, blockIdx.y, tile, lane, n_neg, n_zero);
        }
        return;
    }

    // scalar path: what does not fill a tile, and the zero padding words
    const size_t i = a.n_tiles * (size_t)kCoords + (size_t)(blockIdx.x - a.n_tiles) * kWave + lane;
    const bool in = i < a.d;
    const size_t word = i >> 5;
    const bool writes_word = (lane & 31) == 0 && word < a.words_total;
    int n_neg = 0, n_zero = 0;
    for (int w = VOTE ? 0 : (int)blockIdx.y; w < (VOTE ? M : (int)blockIdx.y + 1); ++w) {
        float v = 0.0f;
        if (in) {
            v = G::load1(a.g[w], i);
            if (HAS_M) {
                v = momentum(a.beta, a.omb, a.m[w][i], v);
                a.m[w][i] = v;
            }
        }
        const bool abstain = in && __builtin_fabsf(v) < a.tau;
        const bool neg = in && !abstain && v < 0.0f;
        n_neg += neg ? 1 : 0;
        n_zero += abstain ? 1 : 0;
        if (!VOTE) {
            const uint64_t nmask = __builtin_amdgcn_ballot_w64(neg);
            const uint64_t zmask = __builtin_amdgcn_ballot_w64(abstain);
            if (writes_word) {
                a.neg_out[w * a.plane_stride + word] = (uint32_t)(lane == 0 ? nmask : nmask >> 32);
                a.zero_out[w * a.plane_stride + word] = (uint32_t)(lane == 0 ? zmask : zmask >> 32);
            }
        }
    }
    if (VOTE) {
        const uint32_t ans = in ? quorum_answer(n_neg, n_zero, M, a.quorum) : 0u;
        if (in) a.x[i] = step_ternary(a.x[i], a.delta, ans);
        const uint64_t nmask = __builtin_amdgcn_ballot_w64((ans & 1u) != 0);
        const uint64_t zmask = __builtin_amdgcn_ballot_w64((ans & 2u) != 0);
        if (writes_word) {
            a.voted_neg[word] = (uint32_t)(lane == 0 ? nmask : nmask >> 32);
            a.voted_zero[word] = (uint32_t)(lane == 0 ? zmask : zmask >> 32);
        }
    }
}

// ----------------------------------------------------------- server ----

struct QuorumVoteArgs {
    const uint32_t *neg[64];
    const uint32_t *zero[64];
    uint32_t *voted_neg;
    uint32_t *voted_zero;
    int M;
    int quorum;
    size_t d;
    size_t n_vec;     // 128-bit groups of words, padding included
};

// Bit-sliced, like the binary vote: a lane holds 128 coordinates (four words)
// of every plane.  The numbers of "-" votes (n) and of abstentions (z) are
// counted into binary planes, a batch of workers at a time; then
// t = 2 n + z is formed plane by plane, and since S = #plus - #minus = M - t,
//     answer "-"  iff  S <= -Q  iff  t >= M + Q
//     answer  0   iff  |S| < Q  iff  M - Q < t < M + Q
// which are two comparisons of t with constants, done from the lowest plane up.
__device__ __forceinline__ u32x4 splat(uint32_t v) { return u32x4{v, v, v, v}; }

// planes of (t >= c) for a constant c, t given by its N binary planes
template <int N>
__device__ __forceinline__ u32x4 planes_ge(const u32x4 (&t)[N], int c) {
    if (c <= 0) return splat(0xFFFFFFFFu);
    if (c >= (1 << N)) return splat(0u);
    u32x4 ge = splat(0xFFFFFFFFu);
#pragma unroll
    for (int k = 0; k < N; ++k) ge = ((c >> k) & 1) ? (t[k] & ge) : (t[k] | ge);
    return ge;
}

// NB workers' planes loaded together (no test between the loads), then counted
template <int P, int NB, typename At>
__device__ __forceinline__ void quorum_batch(const uint32_t *const *neg, const uint32_t *const *zero, const At &at,
                                             u32x4 (&n)[P], u32x4 (&z)[P]) {
    u32x4 nw[NB], zw[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        nw[j] = at.load(neg[j]);
        zw[j] = at.load(zero[j]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NB; ++j) nw[j] &= ~zw[j];   // an abstention is not a vote, whatever the other plane says
    add_words<0>(n, nw);
    add_words<0>(z, zw);
}

// the m <= NMAX workers that the full batches leave over, as one batch of exactly that size
template <int P, int NMAX, typename At>
__device__ __forceinline__ void quorum_rest(const uint32_t *const *neg, const uint32_t *const *zero, int m, const At &at,
                                            u32x4 (&n)[P], u32x4 (&z)[P]) {
    if (m == NMAX) {
        quorum_batch<P, NMAX>(neg, zero, at, n, z);
    } else if constexpr (NMAX > 1) {
        quorum_rest<P, NMAX - 1>(neg, zero, m, at, n, z);
    }
}

// P = number of binary planes of n and z (M < 2^P); t = 2 n + z <= 2 M needs one more.
// HOLD_KB: LDS reserved to cap the blocks per compute unit; NB: workers (two planes each) whose words are loaded together.
template <int P, int BLOCK, int HOLD_KB, uint32_t CHUNK, int NB>
__global__ __launch_bounds__(BLOCK) void quorum_vote_kernel(const QuorumVoteArgs a) {
    reserve_lds<HOLD_KB>(a.d == ~(size_t)0, a.voted_neg);
    constexpr int kCountPlanes = P;
    constexpr int kTotalPlanes = P + 1;
    const Group<CHUNK, BLOCK> at(a.n_vec);
    const size_t u = at.u;
    if (u >= a.n_vec) return;
    u32x4 n[kCountPlanes], z[kCountPlanes];
#pragma unroll
    for (int k = 0; k < kCountPlanes; ++k) n[k] = z[k] = splat(0u);
    int w0 = 0;
    for (; w0 + NB <= a.M; w0 += NB) quorum_batch<P, NB>(a.neg + w0, a.zero + w0, at, n, z);
    quorum_rest<P, NB - 1>(a.neg + w0, a.zero + w0, a.M - w0, at, n, z);
    // t = 2 n + z
    u32x4 t[kTotalPlanes];
    t[0] = z[0];
    u32x4 carry = splat(0u);
#pragma unroll
    for (int k = 1; k < kTotalPlanes; ++k) {
        const u32x4 x = k - 1 < kCountPlanes ? n[k - 1] : splat(0u);
        const u32x4 y = k < kCountPlanes ? z[k] : splat(0u);
        const u32x4 xy = x ^ y;
        t[k] = xy ^ carry;
        carry = (x & y) | (xy & carry);
    }
    const u32x4 is_neg = planes_ge(t, a.M + a.quorum);
    const u32x4 not_plus = planes_ge(t, a.M - a.quorum + 1);
    u32x4 live;
    live.x = live_mask(4 * u + 0, a.d);
    live.y = live_mask(4 * u + 1, a.d);
    live.z = live_mask(4 * u + 2, a.d);
    live.w = live_mask(4 * u + 3, a.d);
    st_stream(reinterpret_cast<u32x4 *>(a.voted_neg) + u, is_neg & live);
    st_stream(reinterpret_cast<u32x4 *>(a.voted_zero) + u, not_plus & ~is_neg & live);
}

// The decision for one word of coordinates: neg_at(w) and zero_at(w) are where worker w's words lie, NB
// workers' two words are out together.  As quorum_vote_kernel: counts n and z in P planes, t = 2 n + z
// against M + Q and M - Q + 1 from the lowest plane up.
template <int P, int NB, typename At1, typename At2>
__device__ __forceinline__ void quorum_word(At1 neg_at, At2 zero_at, int M, int Q, uint32_t &is_neg, uint32_t &not_plus) {
    uint32_t n[P], z[P];
#pragma unroll
    for (int k = 0; k < P; ++k) n[k] = z[k] = 0;
    for (int w0 = 0; w0 < M; w0 += NB) {
        uint32_t nw[NB], zw[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int w = w0 + j < M ? w0 + j : w0;
            nw[j] = *neg_at(w);
            zw[j] = *zero_at(w);
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            nw[j] = w0 + j < M ? nw[j] & ~zw[j] : 0u;   // an abstention is not a vote
            zw[j] = w0 + j < M ? zw[j] : 0u;
        }
        add_words<0>(n, nw);
        add_words<0>(z, zw);
    }
    is_neg = not_plus = 0xFFFFFFFFu;
    uint32_t carry = 0;
    const int hi = M + Q, lo = M - Q + 1;
#pragma unroll
    for (int k = 0; k <= P; ++k) {
        const uint32_t u = k > 0 ? n[k > 0 ? k - 1 : 0] : 0u, v = k < P ? z[k < P ? k : 0] : 0u;
        const uint32_t uv = u ^ v, t = uv ^ carry;
        carry = (u & v) | (uv & carry);
        is_neg = ge_step(is_neg, t, hi, k);
        not_plus = ge_step(not_plus, t, lo, k);
    }
    if (hi >= (2 << P)) is_neg = 0u;           // t < 2^(P + 1)
    if (lo <= 0) not_plus = 0xFFFFFFFFu;
}

// The server's answer for a vector of a few million coordinates: one word a lane (see vote_word_kernel)
template <int P>
__global__ __launch_bounds__(64) void quorum_word_kernel(const QuorumVoteArgs a) {
    const size_t wi = (size_t)blockIdx.x * 64 + threadIdx.x;
    if (wi >= 4 * a.n_vec) return;
    uint32_t is_neg, not_plus;
    quorum_word<P, 8>([&](int w) { return a.neg[w] + wi; }, [&](int w) { return a.zero[w] + wi; }, a.M, a.quorum, is_neg, not_plus);
    const uint32_t live = live_mask(wi, a.d);
    a.voted_neg[wi] = is_neg & live;
    a.voted_zero[wi] = not_plus & ~is_neg & live;
}

// ----------------------------------------------------- server + apply ----
// The answer and the update in one launch, from planes that one pack launch over all workers left in
// memory (vote_apply_kernel's counterpart): a lane decides a word's 32 coordinates, LDS hands the
// two words of the answer to the lanes that own x.

struct QuorumApplyArgs {
    const uint32_t *neg;      // worker 0's planes; the next worker's lie plane_stride words further
    const uint32_t *zero;
    size_t plane_stride;
    uint32_t *voted_neg;
    uint32_t *voted_zero;
    float *x;
    float delta;
    int M;
    int quorum;
    size_t d;
    size_t words_total;
};

// P planes of the counts, as quorum_vote_kernel.  A block owns R rows of 1024 coordinates.
template <int P, int NB, int R, int HOLD_KB>
__global__ __launch_bounds__(kBlock) void quorum_apply_kernel(const QuorumApplyArgs a) {
    reserve_lds<HOLD_KB>(a.d == ~(size_t)0, a.voted_neg);
    constexpr int kWords = 32 * R;
    __shared__ uint32_t answer[2][kWords];
    const int tid = threadIdx.x;
    const size_t wi = (size_t)blockIdx.x * kWords + tid;
    const size_t base = (size_t)blockIdx.x * (R * kRowCoords);
    const bool full = base + (size_t)(R * kRowCoords) <= a.d;
    f32x4 xv[R];
    const Window xw = window(a.x, base * sizeof(float), full ? R * kRowCoords * sizeof(float) : 0);
#pragma unroll
    for (int r = 0; r < R; ++r) xv[r] = ld_quad(xw, (r * kBlock + tid) * 16);
    if (tid < kWords && wi < a.words_total) {
        uint32_t is_neg, not_plus;
        quorum_word<P, NB>([&](int w) { return a.neg + w * a.plane_stride + wi; },
                                     [&](int w) { return a.zero + w * a.plane_stride + wi; }, a.M, a.quorum, is_neg, not_plus);
        const uint32_t live = live_mask(wi, a.d);
        const uint32_t neg = is_neg & live, zero = not_plus & ~is_neg & live;
        a.voted_neg[wi] = neg;
        a.voted_zero[wi] = zero;
        answer[0][tid] = neg;
        answer[1][tid] = zero;
    }
    __syncthreads();
    if (full) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int word = r * 32 + (tid >> 3), shift = (tid & 7) * 4;
            const uint32_t nn = answer[0][word] >> shift, zn = answer[1][word] >> shift;
            f32x4 v = xv[r];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = step_ternary(v[c], a.delta, ((nn >> c) & 1u) | (((zn >> c) & 1u) << 1));
            st_quad<kThrough>(xw, (r * kBlock + tid) * 16, v);
        }
        return;
    }
    for (int i = tid; base + i < a.d; i += kBlock) {
        const uint32_t ans = ((answer[0][i >> 5] >> (i & 31)) & 1u) | (((answer[1][i >> 5] >> (i & 31)) & 1u) << 1);
        a.x[base + i] = step_ternary(a.x[base + i], a.delta, ans);
    }
}

// ------------------------------------------------------------ apply ----

struct TernaryApplyArgs {
    float *x;
    const uint32_t *neg;
    const uint32_t *zero;
    float delta;
    uint32_t n_tiles;
    size_t d;
};

// in the shapes of apply_kernel
template <bool SMALL>
__global__ __launch_bounds__(kWave) void ternary_apply_kernel(const TernaryApplyArgs a) {
    using S = ApplyShape<SMALL>;
    const uint32_t lane = threadIdx.x;
    if (blockIdx.x < a.n_tiles) {
        const size_t tile = die_tile<S::kChunk>(blockIdx.x, a.n_tiles);
        const size_t first = tile * (S::kCoords / 32);
        const Window xw = window(a.x, tile * (S::kCoords * sizeof(float)), S::kCoords * sizeof(float));
        f32x4 xv[S::kRows];
        uint32_t nw[S::kRows], zw[S::kRows];
#pragma unroll
        for (int r = 0; r < S::kRows; ++r) {
            nw[r] = a.neg[first + ((r * kWave + lane) >> 3)];
            zw[r] = a.zero[first + ((r * kWave + lane) >> 3)];
            xv[r] = ld_quad(xw, (r * kWave + lane) * 16);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < S::kRows; ++r) {
            const uint32_t nn = nw[r] >> ((lane & 7) * 4), zn = zw[r] >> ((lane & 7) * 4);
            f32x4 v = xv[r];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = step_ternary(v[c], a.delta, ((nn >> c) & 1u) | (((zn >> c) & 1u) << 1));
            st_quad<S::kStore>(xw, (r * kWave + lane) * 16, v);
        }
        return;
    }
    const size_t i = a.n_tiles * (size_t)S::kCoords + (size_t)(blockIdx.x - a.n_tiles) * kWave + lane;
    if (i < a.d) {
        const uint32_t ans = ((a.neg[i >> 5] >> (i & 31)) & 1u) | (((a.zero[i >> 5] >> (i & 31)) & 1u) << 1);
        a.x[i] = step_ternary(a.x[i], a.delta, ans);
    }
}

}  // namespace ss
