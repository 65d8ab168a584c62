// C ABI of the library (see include/signsgd.h): argument validation, kernel
// selection and launch.  Nothing here allocates or synchronises.
#include "../../include/signsgd.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "step_kernels.hpp"
#include "vote_apply_kernels.hpp"
#include "stats_kernels.hpp"
#include "ternary_kernels.hpp"

// Scratch area of ss_density_static: the same layout ss_density finds in its caller's workspace,
// one copy per device that loads this library, zero when the module is loaded and left zero
// (ticket) by every call that runs to completion.  In host code this name only stands for the
// symbol; the device address comes from hipGetSymbolAddress (see ss_density_static).
static __device__ __align__(256) unsigned long long scratch[sizeof(ss::DensityScratch) / sizeof(unsigned long long)];

namespace {

thread_local int g_last_hip_error = 0;

// device address of `scratch` on each device, looked up the first time a device is used
constexpr int kMaxDevices = 64;
std::atomic<ss::DensityScratch *> g_scratch_on_device[kMaxDevices];

constexpr size_t kMaxGrid = 0x7FFFFFFFull;

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline size_t grad_bytes(ss_dtype gdt) { return gdt == SS_BF16 ? 2 : 4; }

// binary digits needed for a count of up to M votes
inline int count_planes(int M) {
    int p = 1;
    while ((1 << p) <= M) ++p;
    return p;
}

// A buffer of one call, for the check that nothing that is written shares a byte
// with anything else (buffers that are only read may coincide, e.g. one gradient
// handed in for two workers).
struct Span {
    uintptr_t lo, hi;   // [lo, hi); empty spans (NULL pointer or no bytes) never overlap
    bool written;
};

inline Span span(const void *p, size_t bytes, bool written) {
    const uintptr_t lo = reinterpret_cast<uintptr_t>(p);
    return Span{lo, p ? lo + bytes : lo, written};
}

// sorts s; true iff a written span overlaps any other span
inline bool written_spans_overlap(Span *s, int n) {
    std::sort(s, s + n, [](const Span &a, const Span &b) { return a.lo < b.lo; });
    uintptr_t end_any = 0, end_written = 0;   // furthest end among the spans seen so far
    for (int i = 0; i < n; ++i) {
        if (s[i].lo == s[i].hi) continue;
        if (s[i].lo < (s[i].written ? end_any : end_written)) return true;
        end_any = std::max(end_any, s[i].hi);
        if (s[i].written) end_written = std::max(end_written, s[i].hi);
    }
    return false;
}

// Every kernel takes one argument struct by value.  The status is the launch
// call's own return value: an error left on this thread by an earlier, unrelated
// runtime call is neither reported as ours nor cleared.
template <typename Args>
int launch(void (*kernel)(Args), size_t grid, unsigned lds_bytes, hipStream_t stream, const Args &a,
           int block = ss::kBlock, int grid_y = 1) {
    void *params[1] = {const_cast<Args *>(&a)};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3((unsigned)grid, (unsigned)grid_y),
                                         dim3((unsigned)block), params, lds_bytes, stream);
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        return SS_ERR_HIP;
    }
    return SS_OK;
}

// how the coordinate range is cut for a kernel that handles R rows per block
struct Tiling {
    size_t n_tiles;      // blocks on the vector path
    size_t tail_blocks;  // blocks of kBlock scalar coordinates, zero padding included
    size_t words_total;
};

inline Tiling make_tiling(size_t d, int rows, bool covers_padding, int block = ss::kBlock, int per_lane = ss::kQuad) {
    Tiling t;
    const size_t tile = (size_t)rows * block * per_lane;
    t.words_total = ss_packed_bytes(d) / 4;
    t.n_tiles = d / tile;
    const size_t done = t.n_tiles * tile;
    const size_t end = covers_padding ? t.words_total * 32 : d;
    t.tail_blocks = (end - done + block - 1) / block;
    return t;
}

// ------------------------------------------------------------------------
// Launch shapes of the step kernel (see step_kernels.hpp for the reasoning).
//   streaming shape, several workers and more bytes than the line below: one or a few workers at a time, and a
//     reservation of LDS that no kernel touches, sized so that the wanted number of blocks fits in the 160 KB of a
//     gfx950 compute unit (the only one that the library is built for)
//   latency shape, everything smaller: the loads of up to eight workers at once, no cap
// The line between them, in bytes of gradients and momentum, where momentum counts twice, read and written, here and below.  With momentum it is
// 5 x 2^25, us, latency / streaming with x kept (kKeepX), the same state again and twelve and more in turn: M = 2 7.2 M coordinates 37.3 / 34.4 and 38.8 / 37.5, M = 4 3.6 M
// 33.3 / 31.5 and 34.7 / 32.5, M = 7 2.05 M 32.2 / 31.3 and 34.0 / 33.2, 2.8 M 45.0 / 42.8 and 45.5 / 43.0, M = 12 1.2 M 31.7 / 29.7 and 33.8 / 31.2, M = 16 900,000 32.3 / 33.4
// and 34.3 / 34.5, 1.3 M 46.7 / 43.0 and 48.1 / 43.2, bf16 M = 8 2.2 M 33.0 / 32.8 and 35.0 / 35.0, M = 16 1.3 M 37.7 / 35.8 and 40.8 / 37.4.  Without momentum it is 2^28.
// The latency shape with all lines kept (kKeep) is faster on the far side as long as nothing else comes between the steps, and slower as soon as
// something does.  us, kept / streaming, one state, three in turn, twelve and more, and one state behind a 600 MB copy (copy and step): M = 4 4.4 M 36.3 / 39.0, 36.9 / 39.2,
// 44.6 / 39.4, 155.0 / 152.9; M = 7 2.2 M 29.9 / 33.4, 31.4 / 34.4, 38.6 / 34.7, 149.7 / 147.4; M = 16 1.1 M 34.8 / 37.6, 35.4 / 37.5, 44.0 / 37.6, 155.3 / 150.1; M = 33 650,000
// 41.1 / 42.7, 43.1 / 42.9, 54.1 / 42.9, 164.6 / 154.6.
// Below the line the latency shape leaves its lines to the L2 with nt.  Kept as well, from some 16 MB written on, us, to the L2 / kept: one state M = 7 700,001 10.0 / 10.5,
// 1.5 M 23.1 / 19.8, M = 4 1.2 M 10.3 / 10.4, M = 16 600,000 19.6 / 18.3, three in turn 12.0 / 11.0, 25.4 / 22.1, 12.5 / 11.4, 22.1 / 22.4, twelve and more 12.7 / 14.9,
// 26.0 / 27.7, 13.1 / 14.6, 22.7 / 27.5, M = 64 150,000 25.4 / 25.8, 27.3 / 34.0, 32.9 / 44.9, M = 1 4.0 M 12.1 / 10.5, 13.7 / 12.7, 14.8 / 15.8; gradients alone, where x is all
// that is written, M = 3 5.0 M 14.5 / 13.7, 17.1 / 16.6, 17.7 / 18.9, bf16 M = 8 9.0 M 34.4 / 32.9, 36.4 / 34.7, 37.4 / 40.3; behind a 600 MB copy level in all of them.  A step
// that finds its lines again is one with nothing before it; bucket after bucket, or layer after layer, of a larger model finds none.
// The streaming shapes of the binary step keep the first kKeepX bytes of x, the buffer that the program reads next, without momentum up to eight workers (kKeepXWorkers); so do
// smaller steps of one worker without momentum (one_keeps).  us, nothing kept / 64 MB / 84 MB / all of x, one state again and again: M = 1 without momentum 25.6 M 47.1 / 45.3 /
// 44.5 / 43.9, 138 M 241.4 / 239.6 / 239.2 / 255, with 25.6 M 77.0 / 75.0 / 73.4 / 72.3, M = 2 25.6 M 122.3 / 118.4 / 117.1 / 116.2, bf16 alone M = 8 25.6 M 96.5 / 92.6 / 90.9 /
// 89.5, 18 M 68.6 / 64.5 / 64.0 / 64.0; three states in turn, which is why it is not more: 47.0 / 45.4 / 44.8 / 47.7, 243.0 / 241.6 / 244.1 / 253, 77.0 / 74.2 / 73.0 / 77.6,
// 122.3 / 118.0 / 116.8 / 122.3, 98.7 / 93.6 / 92.3 / 100.7, 69.8 / 64.7 / 64.0 / 64.0.
// That holds for steps that follow one another closely.  Twelve states in turn, and step, a read of x and a 600 MB copy (all three), not / kept: with momentum M = 1 25.6 M 77.9 / 79.1
// and 226.1 / 226.3, M = 2 122.0 / 123.5 and 271.5 / 271.5, M = 4 5.0 M 45.0 / 43.5 and 166.8 / 166.2, M = 7 8.0 M 114.8 / 115.0 and 243.3 / 240.6, bf16 M = 5 25 M 223.2 / 224.9 and
// 372.9 / 371.5; alone M = 1 25.6 M 47.3 / 48.8 and 195.8 / 195.9, M = 3 76.7 / 78.5 and 225.2 / 225.5, M = 7 135.5 / 141.3 and 288.9 / 292.2, bf16 M = 6 25 M 80.0 / 81.9 and 228.4 / 227.7,
// M = 8 25.6 M 98.3 / 101.7 and 246.1 / 248.8.  Above eight workers alone it costs more than it gives: three states, twelve, step and read and copy, M = 9 12 M 84.5 / 81.3, 83.7 / 88.2,
// 219.0 / 219.0, 30 M 197.5 / 194.0, 196.0 / 205.5, 361.4 / 365.4, bf16 M = 16 10 M 67.0 / 66.6, 68.9 / 73.1, 199.5 / 199.1, M = 24 9 M 85.1 / 83.0, 89.5 / 94.8, 218.0 / 218.1.
// Vote and update gain nothing (M = 8 bf16 6.6 M with the bits 90.9 / - / 90.1, M = 12 8.8 M 203 / - / 203), the ternary step loses (launch_ternary).
// Without momentum, where x alone is written, the streaming shapes pay from 2^28 bytes of gradients on.
constexpr size_t kKeepX = (size_t)9 << 23;
constexpr int kKeepXWorkers = 8;
// Tiles of x that are kept: none in a step that moves 2^31 bytes or more, where what is kept no longer waits for the next step but costs its way out, us without /
// with 75 MB: M = 1 300 M 876 / 885, bf16 alone M = 2 380 M 672 / 682; below M = 1 alone 138 M 241.6 / 240.5, M = 2 60 M 282.5 / 279.1.
inline uint32_t x_tiles_kept(int M, size_t d, size_t worker_bytes, size_t tile_bytes) {
    return d * (M * worker_bytes + 2 * sizeof(float)) < (size_t)1 << 31 ? (uint32_t)(kKeepX / tile_bytes) : 0;
}
// One worker streams from 11 x 2^23 bytes of momentum and x written on (x alone where there is no momentum): us, to the L2 / streaming with x kept, three states in turn, with
// momentum 13 M 42.7 / 38.3, twelve 43.0 / 42.6.  Without momentum x is kept below as well, in the shape of the smaller steps, from 24 MB of it on (bf16 48): to the L2 / kept, one
// state, three, a dozen and more, and step, a read of x and a 600 MB copy: 6.4 M 11.3 / 10.4, 12.7 / 12.7, 14.0 / 14.6, 137.5 / 137.1; 12 M 21.2 / 19.5, 23.1 / 21.9, 23.9 / 24.5,
// 154.9 / 153.2; bf16 12.8 M 19.6 / 17.4, 21.2 / 19.4, 21.7 / 22.1, 153.5 / 152.8; against streaming 20 M 37.9 / 34.6, 38.0 / 35.0, 38.0 / 38.9, 179.8 / 178.2.
constexpr size_t kOneWorkerStreams = (size_t)11 << 23;
inline bool one_streams(size_t d, bool has_m) { return d * sizeof(float) * (has_m ? 2 : 1) >= kOneWorkerStreams; }
inline bool one_keeps(size_t d, bool bf16) { return d * sizeof(float) >= (size_t)(bf16 ? 6 : 3) << 23; }
constexpr size_t kStreams = (size_t)5 << 25;    // with momentum
inline bool streams(int M, size_t d, bool has_m, size_t worker_bytes) {
    return d * (size_t)M * worker_bytes >= (has_m ? kStreams : (size_t)1 << 28);
}

// Given packed_out buffers, the step runs as two launches - pack_kernel over all workers, then vote
// and update - from here on.  A one-pass kernel keeps 2M + 1 buffers open; the two launches stream three at a time, but
// cost a second launch and tail (~2.5 us) and read the bits again.  One pass / two launches, us, bytes of gradients and
// momentum: M = 2 fp32 8.8 M 45.1 / 48.7, 25.6 M 124.7 / 125.6, 60 M 287 / 290; M = 3 8.8 M 61.5 / 63.7, 25.6 M (920 MB)
// 171.1 / 170.4, bf16 8.8 M 54.2 / 57.5, 138 M (4.2 GB) 802 / 787; M = 4 17.6 M (845 MB) 149.2 / 149.6, 25.6 M (1.2 GB) 217 / 214;
// M = 5 8.8 M (528 MB) 94.0 / 94.3, 25.6 M (1.5 GB) 265 / 260; M = 7 2.2 M (185 MB) 35.4 / 35.4, 4.4 M (370 MB) 65.1 / 64.9, 6.6 M
// 95.6 / 93.3; M = 9 1.1 M (119 MB) 23.1 / 24.0; M = 16 1.1 M (211 MB) 38.8 / 37.7; bf16 M = 8 4.4 M 65.5 / 62.1.  Up to the next
// step of the rule M = 6 and 7 differ by type: 268 MB fp32 49.0 / 49.8 and 47.8 / 49.9, bf16 51.8 / 50.9 and 51.6 / 49.8, 537 MB
// fp32 94.4 / 94.2 and 91.8 / 92.8, bf16 98.1 / 93.7 and 96.8 / 94.4.  From eight workers on one pass with its lines kept is faster up to 92 MB written
// as long as nothing else comes between the steps, twelve states in turn it is not: M = 8 1.6 M 25.0 / 28.5 and 33.4 / 30.1, 2.5 M 39.9 / 42.2 and 51.0 / 45.4, M = 16 1.1 M 35.1 /
// 36.6 and 44.4 / 38.1, bf16 M = 8 2.4 M 32.9 / 35.8 and 41.8 / 39.0.
// Without momentum where the streaming shapes begin, bytes of gradients: fp32 M = 2 8.4 M (67 MB) 22.7 / 27.2, 33.5 M (268 MB) 83.2 /
// 86.8 before the line and 92.3 / 88.4 behind it, 67 M 183 / 166, M = 4 4.2 M 17.6 / 21.8, 16.8 M 66.6 / 67.0, 33.6 M 122.4 / 125.1,
// 134 M 503 / 493, M = 8 4.2 M 29.6 / 32.3, 8.4 M 57.7 / 58.1 and 61.7 / 57.0, 16.8 M 116 / 106, M = 16 4.2 M 53.2 / 54.2, 7.8 M
// 111.8 / 93.0; bf16 M = 3 5.6 M 14.9 / 18.3, 41.7 M (250 MB) 91.7 / 94.5, M = 8 4.2 M 19.3 / 24.5, 15.7 M 64.3 / 65.6.
// step_bf16_kernel, which writes no bits, starts at the same line.
inline bool split_pays(int M, size_t d, bool has_m, size_t worker_bytes) {
    if (M < 2 || d < ((size_t)1 << 20)) return false;
    if (!has_m) return streams(M, d, false, worker_bytes);
    return M >= 3 && d * (size_t)M * worker_bytes >= ((size_t)1 << (M >= 8 ? 27 : M >= 6 ? 28 : 30));
}

// A launch may have at most 2^32 - 1 threads, which a shape with one row of quads a lane reaches at 2^34
// coordinates.  Up to half of that every shape is safe, the blocks of a tail included; a step over a longer vector
// runs over parts of this many coordinates, the ternary step and sigma take two rows there, and the other calls end
// at the limit itself.
constexpr size_t kOneRowMaxD = (size_t)1 << 33;
// no step is longer (nor fits: 4 bytes of x alone are 275 GB)
constexpr size_t kStepMaxD = (size_t)1 << 36;

// With lent scratch memory the step takes the same two launches without packed_out, over slabs of the
// vector whose bits fit into it.  kScratchBytes bounds what is asked for: at M = 16 a slab of 67 M
// coordinates, 2 ms of work for each further pair of launches (~5 us).
constexpr size_t kScratchBytes = (size_t)128 << 20;
constexpr size_t kScratchMinSlab = (size_t)1 << 20;

// coordinates of a slab: all d if the bits of M workers fit into `bytes` (and one launch), otherwise equal parts of a
// multiple of 8192 (every buffer's part stays 16-byte aligned); 0 if there is no room for 8192
inline size_t scratch_slab(int M, size_t d, size_t bytes) {
    if (d <= kOneRowMaxD && (size_t)M * ss_packed_bytes(d) <= bytes) return d;
    const size_t room = std::min(bytes / (size_t)M * 8 / 8192 * 8192, kOneRowMaxD);
    if (room == 0) return 0;
    const size_t parts = (d + room - 1) / room;
    return std::min(room, ((d + parts - 1) / parts + 8191) / 8192 * 8192);
}

// One pass / two launches with scratch, us behind queued work, MB of gradients and momentum: fp32 M = 4 805 MB 144 / 142, 1,074 188 /
// 189, 2,147 372 / 369; M = 5 268 48.3 / 51.0, 537 93.4 / 93.9, 805 140 / 140, 1,074 186 / 183; M = 6 537 92.9 / 94.4, 805 137 / 137, 2,147
// 359 / 357; M = 7 268 47.0 / 49.1, 537 90.4 / 93.1, 805 136 / 135, 2,147 354 / 352; M = 8 268 48.6 / 48.6, 403 70.7 / 69.1, 805 137 / 133;
// M = 12 403 70.9 / 68.3; M = 16 268 51.5 / 48.5, 138 M 4,520 / 4,060; bf16 M = 4 1,074 195 / 193, 2,147 390 / 384; M = 5 537 97.6 / 98.0,
// 805 146 / 141; M = 7 537 94.0 / 94.2, 805 140 / 137; M = 8 268 48.4 / 49.1, 524 94 / 90; M = 12 268 51.9 / 47.0.  Three workers
// 389 / 387 at 2,147 MB, two 424 / 422 (bf16 444 / 447): never.  The step with abstentions takes the same lines: M = 4 1,074 191 / 192,
// bf16 2,147 388 / 395, M = 7 805 138 / 137, M = 8 268 47.6 / 50.1, 403 70.5 / 69.7, bf16 268 51.2 / 50.1, M = 16 805 136 / 129.
// A lender that asks the device for its free memory at each call, borrows and launches twice spends 10-15 us of host time on it,
// which queued work hides: waited for after each step M = 5 268 MB takes 74.5 us where one pass takes 59.5, 1,080 MB 209 / 196.
inline bool scratch_pays(int M, size_t d, size_t worker_bytes) {
    const int many = worker_bytes < 12 ? 5 : 6;    // bf16, fp32
    return M >= 4 && d * (size_t)M * worker_bytes >= (size_t)(M >= 8 ? 1 : M >= many ? 3 : 4) << 28;
}

// any-M vote and update, and answer and update: from about a gigabyte of x on, one row per block is 3-7 % faster than four
constexpr size_t kLargeD = (size_t)1 << 28;

// the updates alone (see ApplyShape): two rows a wave up to here
constexpr size_t kApplySmall = (size_t)1 << 23;

template <typename Args>
int launch_apply(void (*small)(Args), void (*large)(Args), Args a, void *hip_stream) {
    const bool two_rows = a.d < kApplySmall || a.d >= kOneRowMaxD;   // beyond, a row a lane has too many threads
    const Tiling t = make_tiling(a.d, two_rows ? 2 : 1, false, ss::kWave);
    const size_t grid = t.n_tiles + t.tail_blocks;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    a.n_tiles = (uint32_t)t.n_tiles;
    return launch(two_rows ? small : large, grid, 0, static_cast<hipStream_t>(hip_stream), a, ss::kWave);
}

template <int NPTR>
void fill_step_args(ss::StepArgs<NPTR> &a, int M, const void *const *g, float *const *m, uint32_t *const *packed,
                    float beta, float delta, float *x, uint32_t *voted, size_t d) {
    for (int w = 0; w < NPTR; ++w) {
        a.p.g[w] = w < M ? g[w] : nullptr;
        a.p.m[w] = (m && w < M) ? m[w] : nullptr;
        a.p.packed[w] = (packed && w < M) ? packed[w] : nullptr;
    }
    a.x = x;
    a.voted = voted;
    a.beta = beta;
    a.omb = 1.0f - beta;
    a.delta = delta;
    a.M = M;
    a.write_packed = packed != nullptr;
    a.warmup = 0;
    a.sum_update = 0;
    a.sums = nullptr;
    a.d = d;
}

template <int MT, int NPTR, int BLOCK, int BW, int R, int HOLD_KB, bool NEAR, int STORE, int STORE_X, uint32_t CHUNK, bool HAS_M, typename G>
int launch_step_shape(ss::StepArgs<NPTR> &a, size_t d, hipStream_t stream) {
    const Tiling t = make_tiling(d, R, true, BLOCK);
    const size_t grid = t.n_tiles + t.tail_blocks;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    a.n_tiles = (uint32_t)t.n_tiles;
    a.x_kept = x_tiles_kept(a.M, d, sizeof(typename G::elem) + (HAS_M ? 2 * sizeof(float) : 0), R * BLOCK * sizeof(ss::f32x4));
    a.words_total = t.words_total;
    // two policies in one kernel cost the sums 3-4 % (M = 3 gradients alone 40 M 121.1 us against 125.0, and see launch_octets)
    if (STORE != STORE_X && (a.x_kept == 0 || a.sums || a.sum_update))
        return launch(ss::step_kernel<MT, NPTR, BLOCK, BW, R, HOLD_KB, NEAR, STORE, STORE, CHUNK, HAS_M, G>, grid, 0, stream, a, BLOCK);
    return launch(ss::step_kernel<MT, NPTR, BLOCK, BW, R, HOLD_KB, NEAR, STORE, STORE_X, CHUNK, HAS_M, G>, grid, 0, stream, a, BLOCK);
}

template <int MT, int NPTR, int BLOCK, int BW, int HOLD_KB, int STORE>
int launch_octets(ss::StepArgs<NPTR> &a, size_t d, hipStream_t stream) {
    const Tiling t = make_tiling(d, 1, true, BLOCK, 2 * ss::kQuad);
    const size_t grid = t.n_tiles + t.tail_blocks;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    a.n_tiles = (uint32_t)t.n_tiles;
    a.x_kept = x_tiles_kept(a.M, d, sizeof(uint16_t), 2 * BLOCK * sizeof(ss::f32x4));
    a.words_total = t.words_total;
    // two policies in one kernel cost the sums 4 % (M = 9 100 M 440 us against 459 with no tile kept)
    if constexpr (MT > 0 && MT <= kKeepXWorkers)
        if (a.x_kept && !a.sums && !a.sum_update) return launch(ss::step_bf16_kernel<MT, NPTR, BLOCK, BW, HOLD_KB, STORE, ss::kKeep>, grid, 0, stream, a, BLOCK);
    return launch(ss::step_bf16_kernel<MT, NPTR, BLOCK, BW, HOLD_KB, STORE, STORE>, grid, 0, stream, a, BLOCK);
}

// what distinguishes the variants of the step (see ss_step_flags)
struct StepVariant {
    unsigned flags;
    int8_t *sums;
};

// MT > 0: M fixed at compile time; MT == 0: any M up to SS_MAX_WORKERS
template <int MT, bool HAS_M, typename G>
int launch_step_m(int M, const void *const *g, float *const *m, uint32_t *const *packed, float beta, float delta,
                  float *x, uint32_t *voted, StepVariant var, size_t d, hipStream_t stream) {
    constexpr int NPTR = MT > 0 ? MT : SS_MAX_WORKERS;
    ss::StepArgs<NPTR> a;
    fill_step_args<NPTR>(a, M, g, HAS_M ? m : nullptr, packed, beta, delta, x, voted, d);
    a.warmup = (var.flags & SS_STEP_WARMUP) ? 1 : 0;
    a.sum_update = (var.flags & SS_STEP_SUM_UPDATE) ? 1 : 0;
    a.sums = var.sums;
    constexpr bool kBf16 = std::is_same<G, ss::Bf16Grad>::value;
    using ss::kKeep;
    using ss::kStream;
    using ss::kThrough;
    if constexpr (MT == 1) {
        // One worker: one-wave blocks; written through and with a cap from one_streams on.  us, as below it /
        // capped / four waves of two rows: with momentum fp32 8.8 M 28.6 / 29.2 / 29.1, 17.6 M 55.8 / 54.7 / 57.2, 25.6 M 79.9 /
        // 77.8 / 82.2, 138 M 433 / 410 / 477, bf16 25.6 M 72.1 / 70.2 / 73.2; without fp32 17.6 M 33.0 / 33.1 / 33.8, 25.6 M
        // 46.8 / 46.8 / 48.3, 60 M 108 / 106 / 116, bf16 138 M 206 / 201 / 226
        if (one_streams(d, HAS_M)) return launch_step_shape<1, NPTR, 64, 1, 1, HAS_M ? 10 : 6, false, kThrough, kKeep, 0, HAS_M, G>(a, d, stream);
        if constexpr (!HAS_M)
            if (one_keeps(d, kBf16)) return launch_step_shape<1, NPTR, 64, 1, 1, 0, true, kKeep, kKeep, 8, false, G>(a, d, stream);
        return launch_step_shape<1, NPTR, 64, 1, 1, 0, true, kStream, kStream, 8, HAS_M, G>(a, d, stream);
    } else {
        constexpr size_t kWorkerBytes = (kBf16 ? 2 : 4) + (HAS_M ? 8 : 0);
        if (streams(M, d, HAS_M, kWorkerBytes)) {
            // Streaming shapes: one-wave blocks of one row, written through, tiles in order.
            if constexpr (HAS_M) {
                // One worker a stage and 10 to 14 waves a unit, the fewer the more workers.  KB held back and us, against the
                // shapes of one to four larger blocks a unit that were used before: fp32 13: 12 M M = 3 82.5 / 87.2, 25.6 M M = 2
                // 122.5 / 134, M = 4 215.6 / 232, 138 M M = 2 647 / 733, M = 4 1,151 / 1,250; 14 (13): M = 5 261.7 (261.8) / 277,
                // M = 9 454.7 (456.9) / 479, M = 16 805 (830) / 840; bf16 11: M = 3 147.2 / 165.6, 138 M M = 2 565 / 674, M = 4 993 / 1,123;
                // 13 (11): M = 7 307.0 (308.9) / 314.9, M = 16 683 (708) / 696, 60 M M = 8 822 (830) / 860.  Runs of tiles a die: 5-10 %
                // slower in each.
                constexpr int kHold = (MT > 0 && MT < 5 ? 13 : 14) - (kBf16 ? (MT > 0 && MT < 5 ? 2 : 1) : 0);
                return launch_step_shape<MT, NPTR, 64, 1, 1, kHold, false, kThrough, kKeep, 0, true, G>(a, d, stream);
            } else if constexpr (kBf16) {
                // step_bf16_kernel: the workers' loads out together, eight at most, fewer blocks per unit the more loads
                // each has out.  us, 25.6 M unless said: M = 2 138 M 248 / 296 (four-wave blocks of two rows before), M = 3 60 M 126.8 /
                // 145.9, M = 4 63.2 / 65.0, 7 86.8, 8 96.3, 12 128, 16 160.7.  x left to the L2 / written through: M = 4 67 M 166 / 159,
                // 134 M 331 / 322, M = 5 54 M 147 / 147, M = 7 38 M 132 / 133, 153 M 510 / 520, M = 8 34 M 128 / 129; beyond eight within 2 %
                // either way, M = 9 30 M 126 / 123, M = 16 9.4 M 64.0 / 64.7, 34 M 211 / 210.
                if constexpr (MT > 0 && MT <= 6) return launch_octets<MT, NPTR, 64, 8, MT == 2 ? 10 : MT == 3 ? 13 : 16, kThrough>(a, d, stream);
                else return launch_octets<MT, NPTR, 64, 8, MT == 16 ? 24 : 20, kStream>(a, d, stream);
            } else {
                // fp32: four workers a stage make up for the missing momentum stream.  us, against two four-wave blocks a unit before:
                // 25.6 M M = 3 76.4 / 83.1, 4 91.8 / 94.6, 7 135.4 / 145.5, 8 153.8 / 160.1, 9 169.0 / 178.3, 16 279.8 / 288.5, 138 M
                // M = 2 319 / 345, M = 7 734 / 806
                return launch_step_shape<MT, NPTR, 64, 4, 1, MT == 2 ? 11 : 13, false, kThrough, (MT > 0 && MT <= kKeepXWorkers ? kKeep : kThrough), 0, false, G>(a, d, stream);
            }
        }
        // Latency shape: the loads of up to eight workers go out together, nothing is held back, buffers are addressed
        // without arithmetic, a die takes runs of 64 (from 2^20 coordinates on 256) tiles.  us, against descriptors / no runs: 10,007 M = 16
        // 3.2 / 3.4 / 3.2, 272,474 M = 7 5.8 / 6.1 / 6.7, M = 16 11.2 / 11.4 / 15.4, M = 9 7.2 / 7.2 / 8.3, 700,001 M = 7 12.4 / 12.6 /
        // 13.3, 1.1 M M = 7 (runs of 256) 18.4 / 18.6 / 19.6, M = 16 38.8 / 38.8 / 43.7, 4.4 M M = 4 - / 42.1 / 44.3, gradients alone
        // 272,474 M = 16 6.0 / 6.0 / 6.5, 8.8 M M = 4 34.3 / 34.2 / 35.6
        constexpr int BW = MT > 0 && MT < 8 ? MT : 8;
        // Written lines that stay in every cache (26 MB in all, up to seven workers, whose loads are one stage) lose: us, the same state again / three
        // in turn / a hundred, to the L2 with nt against without: M = 7 272,474 4.7 / 5.4 / 6.2 against 4.7 / 6.0 / 9.5, M = 5 400,001 4.6 / 5.6 / 6.3 against
        // 4.6 / 6.1 / 8.9, M = 3 700,001 4.9 / 6.0 / 6.7 against 4.9 / 6.4 / 8.0.
        // Sixteen workers with momentum stream before they come to 2^20 coordinates.
        constexpr bool kAlwaysBelow = MT > 0 && HAS_M && MT * kWorkerBytes << 20 >= kStreams;
        if constexpr (!kAlwaysBelow)
            if (d >= ((size_t)1 << 20)) return launch_step_shape<MT, NPTR, 64, BW, 1, 0, true, kStream, kStream, 8, HAS_M, G>(a, d, stream);
        return launch_step_shape<MT, NPTR, 64, BW, 1, 0, true, kStream, kStream, 6, HAS_M, G>(a, d, stream);
    }
}

template <bool HAS_M, typename G>
int launch_step(int M, const void *const *g, float *const *m, uint32_t *const *packed, float beta,
                float delta, float *x, uint32_t *voted, StepVariant var, size_t d, hipStream_t stream) {
#define SS_CASE(n) \
    case n: return launch_step_m<n, HAS_M, G>(M, g, m, packed, beta, delta, x, voted, var, d, stream)
    switch (M) {
        SS_CASE(1); SS_CASE(2); SS_CASE(3); SS_CASE(4); SS_CASE(5); SS_CASE(6); SS_CASE(7); SS_CASE(8);
        SS_CASE(16);
        default: return launch_step_m<0, HAS_M, G>(M, g, m, packed, beta, delta, x, voted, var, d, stream);
    }
#undef SS_CASE
}

// The workers' half of a step: n workers, one launch (see pack_kernel).
template <int NPTR>
int launch_pack_shape(void (*kernel)(ss::PackArgs<NPTR>), ss::PackArgs<NPTR> &a, int n, int block, int rows, int per_lane,
                      hipStream_t stream) {
    const Tiling t = make_tiling(a.d, rows, true, block, per_lane);
    const size_t grid = t.n_tiles + t.tail_blocks;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    a.n_tiles = (uint32_t)t.n_tiles;
    a.words_total = t.words_total;
    return launch(kernel, grid, 0, stream, a, block, n);
}

// Runs of tiles that a die takes at a time (see die_tile): half a megabyte where vectors of up to some tens of millions of
// coordinates are streamed, for in-place kernels that fit the caches a quarter.
//
// With momentum, shapes of pack_kernel (us, fp32 unless said):
//   below 2^28 bytes        written lines left to the L2, quarters.  In order / quarter / half: 17.6 M M = 1 34.2 / 32.6 / 32.9,
//                           4.4 M M = 2 17.7 / 17.4 / 17.4, bf16 17.6 M M = 1 29.0 / 27.4 / 27.8; written through 1.1 M M = 7 16.5
//                           against 15.8
//   up to 2^25 coordinates  written through, halves.  To the L2 in order / to the L2 halves / through in order / through
//                           halves: 25.6 M M = 7 322 / 319 / 320 / 316, M = 1 48.4 / 46.7 / 47.1 / 46.6, 4.4 M M = 8 65.7 / 64.3 /
//                           64.7 / 63.8, bf16 54.8 / 54.1 / 53.8 / 53.3
//   above                   written through, in order, 7 KB held back: 21 waves a unit, 42 KB of loads in flight.  Through halves
//                           without / in order without / in order with: 60 M M = 4 426 / 427 / 421, 138 M M = 4
//                           982 / 986 / 968, 400 M M = 2 1,438 / 1,477 / 1,437, bf16 1,200 / 1,235 / 1,192
template <int NPTR, typename G>
int launch_pack_momentum(ss::PackArgs<NPTR> &a, int n, hipStream_t stream) {
    constexpr size_t kBytes = sizeof(typename G::elem) + 2 * sizeof(float);
    if (a.d * (size_t)n * kBytes < ((size_t)1 << 28))
        return launch_pack_shape(ss::pack_kernel<NPTR, 64, 1, 0, ss::kStream, 8, true, G>, a, n, 64, 1, 4, stream);
    if (a.d < ((size_t)1 << 25))
        return launch_pack_shape(ss::pack_kernel<NPTR, 64, 1, 0, ss::kThrough, 9, true, G>, a, n, 64, 1, 4, stream);
    return launch_pack_shape(ss::pack_kernel<NPTR, 64, 1, 7, ss::kThrough, 0, true, G>, a, n, 64, 1, 4, stream);
}

// Gradients only, one stream that is only read: two rows a wave and half a megabyte a die up to where the runs stop paying,
// which is later in fp32.  In order / in runs, us: fp32 4.4 M M = 8 25.2 / 22.6, 25.6 M M = 1 17.3 / 15.9, M = 7 115 / 111, 60 M
// M = 4 152 / 150, 400 M M = 2 512 / 519; bf16 17.6 M M = 2 13.3 / 12.3, 25.6 M M = 1 9.8 / 9.2, 60 M M = 4 79.6 / 80.2, 138 M
// M = 4 180 / 182.  fp32 beyond 2^27, in order by two waves / in runs, a worker alone 134 M 82.8 / 80.7, 400 M 244.1 / 244.0, 537 M
// 326.7 / 328.5, a step's pack and update M = 4 134 M 493.5 / 495.1, 400 M 1,519 / 1,550, M = 8 200 M 1,290 / 1,317; in order
// by one wave within 0.8 % of two (134 M alone 84.4, otherwise level).
template <int NPTR>
int launch_pack_sign(ss_dtype gdt, ss::PackArgs<NPTR> &a, int n, hipStream_t stream) {
    if (gdt == SS_BF16) {
        if (a.d < ((size_t)1 << 25)) return launch_pack_shape(ss::pack_bf16_kernel<NPTR, 64, 2, 8>, a, n, 64, 2, 8, stream);
        return launch_pack_shape(ss::pack_bf16_kernel<NPTR, 64, 2, 0>, a, n, 64, 2, 8, stream);
    }
    if (a.d < ((size_t)1 << 27))
        return launch_pack_shape(ss::pack_kernel<NPTR, 64, 2, 0, ss::kStream, 8, false, ss::F32Grad>, a, n, 64, 2, 4, stream);
    // two rows a lane have too many threads for the longest vectors
    if (a.d >= kOneRowMaxD)
        return launch_pack_shape(ss::pack_kernel<NPTR, 256, 4, 0, ss::kStream, 0, false, ss::F32Grad>, a, n, 256, 4, 4, stream);
    return launch_pack_shape(ss::pack_kernel<NPTR, 128, 2, 0, ss::kStream, 0, false, ss::F32Grad>, a, n, 128, 2, 4, stream);
}

template <int NPTR>
int launch_pack(int n, const void *const *g, ss_dtype gdt, float *const *m, uint32_t *const *packed, float beta,
                unsigned flags, size_t d, hipStream_t stream) {
    ss::PackArgs<NPTR> a;
    for (int w = 0; w < n; ++w) a.w[w] = ss::PackWorker{g[w], m ? m[w] : nullptr, packed[w]};
    a.beta = beta;
    a.omb = 1.0f - beta;
    a.warmup = (flags & SS_STEP_WARMUP) ? 1 : 0;
    a.d = d;
    if (!m) return launch_pack_sign<NPTR>(gdt, a, n, stream);
    if (gdt == SS_F32) return launch_pack_momentum<NPTR, ss::F32Grad>(a, n, stream);
    return launch_pack_momentum<NPTR, ss::Bf16Grad>(a, n, stream);
}

// Vote and update from packed bits.  A fixed number of workers: blocks of two waves with four rows each, five of them and 40 KB
// of x in flight to a unit.  Both launches of a step against four waves of four rows, three blocks a unit (us): 1.1 M M = 7
// 19.5 / 21.1, 4.4 M 64.8 / 64.2, 25.6 M 348.2 / 351.8, 60 M M = 2 287.4 / 289.8, 138 M M = 4 1,146 / 1,162; one row and no cap:
// 19.7, 64.8, 353, 304, 1,212.  One wave that votes on a word a lane and hands it on by ds_bpermute: 20.6, 67.2, 348.4,
// 287.3, 1,140.
// Any number of workers is added up batch by batch, and the longer a block waits for its votes the more waves a unit
// wants: four waves of four rows, three blocks (count planes four), and from 2^28 coordinates on one row and no cap.
template <int MT, int P>
int launch_vote_apply(const uint32_t *const *packed, int M, uint32_t *voted, float *x, float delta, StepVariant var,
                      size_t d, hipStream_t stream) {
    constexpr int NPTR = MT > 0 ? MT : SS_MAX_WORKERS;
    ss::VoteApplyArgs<NPTR> a;
    for (int w = 0; w < M; ++w) a.packed[w] = packed[w];
    a.voted = voted;
    a.x = x;
    a.sums = var.sums;
    a.delta = delta;
    a.M = M;
    a.sum_update = (var.flags & SS_STEP_SUM_UPDATE) ? 1 : 0;
    a.d = d;
    a.words_total = ss_packed_bytes(d) / 4;
    const size_t words = MT > 0 ? 64 : d >= kLargeD ? 32 : 128;
    const size_t grid = (a.words_total + words - 1) / words;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    if constexpr (MT > 0) return launch(ss::vote_apply_kernel<MT, NPTR, P, 128, 4, 31>, grid, 0, stream, a, 128);
    else if (d >= kLargeD) return launch(ss::vote_apply_kernel<MT, NPTR, P, 256, 1, 0>, grid, 0, stream, a);
    else return launch(ss::vote_apply_kernel<MT, NPTR, P, 256, 4, (P > 0 ? 36 : 40)>, grid, 0, stream, a);
}

int dispatch_vote_apply(const uint32_t *const *packed, int M, uint32_t *voted, float *x, float delta, StepVariant var,
                        size_t d, hipStream_t stream) {
    if (var.sums || (var.flags & SS_STEP_SUM_UPDATE)) {
        const int planes = count_planes(M);
        if (planes <= 3) return launch_vote_apply<0, 3>(packed, M, voted, x, delta, var, d, stream);
        if (planes <= 5) return launch_vote_apply<0, 5>(packed, M, voted, x, delta, var, d, stream);
        return launch_vote_apply<0, 7>(packed, M, voted, x, delta, var, d, stream);
    }
#define SS_CASE(n) \
    case n: return launch_vote_apply<n, 0>(packed, M, voted, x, delta, var, d, stream)
    switch (M) {
        SS_CASE(2); SS_CASE(3); SS_CASE(4); SS_CASE(5); SS_CASE(6); SS_CASE(7); SS_CASE(8);
        SS_CASE(9); SS_CASE(10); SS_CASE(11); SS_CASE(12); SS_CASE(13); SS_CASE(14); SS_CASE(15); SS_CASE(16);
        default: return launch_vote_apply<0, 0>(packed, M, voted, x, delta, var, d, stream);
    }
#undef SS_CASE
}

// the whole step as pack and vote-and-update launches
int launch_two(const void *const *g, ss_dtype gdt, float *const *m, int M, float beta, float delta, float *x,
               uint32_t *voted, uint32_t *const *packed, StepVariant var, size_t d, hipStream_t stream) {
    const int rc = M <= 16 ? launch_pack<16>(M, g, gdt, m, packed, beta, var.flags, d, stream)
                           : launch_pack<SS_MAX_WORKERS>(M, g, gdt, m, packed, beta, var.flags, d, stream);
    if (rc != SS_OK) return rc;
    return dispatch_vote_apply(packed, M, voted, x, delta, var, d, stream);
}

// The votes, sums and quorum votes read M (2 M) buffers at once, in one-wave blocks.  Figures here are over three sets of buffers in
// turn, and one session's differ from another's by 3 %; where a rule was replaced, the figure in brackets is what it gave.  Up to some tens
// of millions of coordinates nothing is held back and a die takes an eighth of a megabyte of every buffer at a time (kVoteChunk); where
// twelve buffers and more are open, from 2^27 coordinates on half a megabyte (kVoteLongChunk) with a cap that leaves fewer waves the
// more loads each has out; from 2^28 on tiles go in order, capped.  us, eighths / halves capped / in order capped: vote M = 7 138 M
// 23.1 / 22.4 / 25.1, M = 9 110 M 23.1 / 23.3 / 24.0, 138 M 28.6 / 27.7 / 28.9, 390 M 78.7 / 75.2 / 75.0; M = 12 100 M 26.6 / - / 28.3, 138 M 36.5 / 35.1 /
// 36.8, M = 16 80 M 28.0 / 28.5 / 30.1, 110 M 38.1 / 38.7 / 39.8, 138 M 47.6 / 46.0 / 50.2, 200 M 68.6 / 66.9 / 69.3, 390 M 134 / 130 / 129, 1,000 M 350 /
// 344 / 327; M = 24 (any) 80 M 40.9 / 40.9 / 42.3, 138 M 70.2 / 67.2 / 72.1, 390 M 198 / 189 / 190, 1,000 M 520 / 508 / 489.  From Python: M = 16
// 138 M 45.5 (48.5), M = 17 110 M 40.5 (43.6), M = 33 138 M 91.1 (97).
constexpr uint32_t kVoteChunk = 7, kVoteLongChunk = 9;
constexpr size_t kVoteRuns = (size_t)1 << 26, kVoteHalves = (size_t)1 << 27, kVoteInOrder = (size_t)1 << 28;

// One word a lane instead of four (the *_word_kernels) up to here; sums and quorum votes of up to eight workers a third of it.  us,
// word / 128-bit lanes: sums M = 16 4.4 M coordinates 4.2 / 5.7, 8.8 M 6.0 / 6.5, 17.6 M 12.7 / 9.9, M = 7 4.4 M 4.0 / 3.7; quorum
// M = 16 8.8 M 7.6 / 8.5, 17.6 M 17.2 / 14.0, M = 3 4.4 M 2.8 / 2.7; vote (more than sixteen workers only) M = 24 4.4 M 5.0 / 5.5, 8.8 M
// 7.1 / 6.6.
constexpr size_t kSumWords = (size_t)3 << 22, kVoteWords = (size_t)3 << 21;
inline bool sum_word_lanes(int M, size_t d) { return d < (M >= 9 ? kSumWords : kSumWords / 3); }

template <int M>
int launch_vote_fixed(const uint32_t *const *packed, uint32_t *voted, size_t d, hipStream_t stream) {
    ss::VoteArgs<M> a;
    for (int w = 0; w < M; ++w) a.packed[w] = packed[w];
    a.voted = voted;
    a.M = M;
    a.d = d;
    a.n_vec = ss_packed_bytes(d) / 16;
    // Up to three workers, little to wait for: four-wave blocks, and from 2^26 coordinates on runs (8.8 M M = 3 2.4 us in runs against 2.3,
    // 25.6 M 3.3 / 3.1, 390 M 30.9 / 31.6).
    const bool few = M < 4 && d < kVoteRuns;
    const size_t block = few ? ss::kBlock : ss::kWave;
    const size_t grid = (a.n_vec + block - 1) / block;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    if constexpr (M < 4) {
        if (few) return launch(ss::vote_kernel<M, ss::kBlock, 0, 0>, grid, 0, stream, a);
        if (d < ((size_t)1 << 34)) return launch(ss::vote_kernel<M, ss::kWave, 0, kVoteChunk>, grid, 0, stream, a, ss::kWave);
        return launch(ss::vote_kernel<M, ss::kWave, 0, 0>, grid, 0, stream, a, ss::kWave);
    } else {
        if (d < (M < 12 ? kVoteInOrder : kVoteHalves)) return launch(ss::vote_kernel<M, ss::kWave, 0, kVoteChunk>, grid, 0, stream, a, ss::kWave);
        if constexpr (M >= 12)
            if (d < kVoteInOrder) return launch(ss::vote_kernel<M, ss::kWave, 20, kVoteLongChunk>, grid, 0, stream, a, ss::kWave);
        return launch(ss::vote_kernel<M, ss::kWave, M >= 8 ? 20 : 8, 0>, grid, 0, stream, a, ss::kWave);
    }
}

int launch_vote_any(const uint32_t *const *packed, int M, uint32_t *voted, size_t d, hipStream_t stream) {
    ss::VoteArgs<SS_MAX_WORKERS> a;
    for (int w = 0; w < SS_MAX_WORKERS; ++w) a.packed[w] = w < M ? packed[w] : nullptr;
    a.voted = voted;
    a.M = M;
    a.d = d;
    a.n_vec = ss_packed_bytes(d) / 16;
    if (d < kVoteWords) return launch(ss::vote_word_kernel, (4 * a.n_vec + 63) / 64, 0, stream, a, 64);
    const size_t grid = (a.n_vec + ss::kWave - 1) / ss::kWave;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    if (d < kVoteHalves) return launch(ss::vote_kernel_any<0, kVoteChunk>, grid, 0, stream, a, ss::kWave);
    if (d < kVoteInOrder) return launch(ss::vote_kernel_any<16, kVoteLongChunk>, grid, 0, stream, a, ss::kWave);
    return launch(ss::vote_kernel_any<16, 0>, grid, 0, stream, a, ss::kWave);
}

// Sums, in runs of 64 tiles a die.  Eight workers' words a batch and the sums written through; from 2^24 coordinates on four to seven
// workers leave them to the L2 and more load four a batch; from kVoteRuns on 7 KB are held back beside the tile's 9, and from eight workers on
// the runs go on to kVoteInOrder.  us, sums to the L2 / through: M = 2 13 M 4.6 / 4.2, 60 M 14.2 / 12.4, M = 7 8.8 M 4.8 / 4.2, 17.6 M 5.8 / 5.6, 25.6 M
// 7.7 / 8.1, 60 M 20.5 / 21.5, M = 16 17.6 M 9.5 / 9.0; eight / four a batch: M = 5 25.6 M 6.7 / 7.3, M = 12 13 M 6.1 / 6.5, 25.6 M 12.0 / 10.9, M = 16
// 25.6 M 14.8 / 12.4, M = 24 13 M 9.8 / 10.0, 17.6 M 13.9 / 13.4, 25.6 M 19.4 / 18.3, 60 M 41.8 / 41.9; beyond, in order / in runs: M = 7 138 M 43.3 / 43.6, M = 9
// 80 M 32.6 / 32.1, M = 12 80 M 35.8 / 34.6, 138 M 57.9 / 56.8, M = 13 138 M 61.1 / 59.5, M = 33 138 M 121.5 / 118, 250 M 211 / 210, M = 24 1,000 M 646 / 652.
// Three sets of buffers in turn, as above; over some fifty, to the L2 / through: M = 3 5.0 M 3.7 / 3.7, 14 M 4.5 / 4.8, 25.6 M 6.2 / 6.7, M = 7 9.0 M 4.9 / 4.8, 14 M 5.6 / 6.2.
template <int P>
int launch_vote_sum(const ss::VoteSumArgs &a, size_t grid, hipStream_t stream) {
    using ss::kStream;
    using ss::kThrough;
    constexpr uint32_t kRun = kVoteChunk - 1;
    if (a.d < kVoteRuns) {
        if (P < 3 || a.d < ((size_t)1 << 24)) return launch(ss::vote_sum_kernel<P, 0, kThrough, kRun, 8>, grid, 0, stream, a, ss::kWave);
        if constexpr (P == 3) return launch(ss::vote_sum_kernel<P, 0, kStream, kRun, 8>, grid, 0, stream, a, ss::kWave);
        else if constexpr (P > 3) return launch(ss::vote_sum_kernel<P, 0, kThrough, kRun, 4>, grid, 0, stream, a, ss::kWave);
    }
    if constexpr (P > 3)
        if (a.d < kVoteInOrder) return launch(ss::vote_sum_kernel<P, 7, kThrough, kRun, 8>, grid, 0, stream, a, ss::kWave);
    return launch(ss::vote_sum_kernel<P, 7, kThrough, 0, 8>, grid, 0, stream, a, ss::kWave);
}

// Quorum votes, us, eighths / halves capped / in order capped: M = 7 80 M 27.3 / 29.9 / 28.2, 138 M 47.6 / 45.0 / 46.2, 390 M 131 / 126 / 121; M = 16
// 80 M 57.6 / 61.3 / 58.4, 110 M 78.5 / - / 79.8, 138 M 100 / 95.0 / 101, 220 M - / 150 / 153, 390 M 282 / 272 / 270; M = 24 110 M 114 / - / 119, 138 M 146 /
// 139 / 146, 220 M - / 220 / 224.  Five to seven workers in halves: 138 M 34.7 (35.8), 39.5 (40.9), 45.0 (45.1), 220 M 53 (52), 61.6 (60.6), 70 (70):
// not worth it.  Up to seven workers in eighths, eight / four a batch, M = 7 17.6 M 7.3 / 7.1, 25.6 M 9.8 / 9.5, 48 M 17.5 / 16.8, M = 6 48 M 15.3 / 14.6,
// M = 5 17.6 M 5.9 / 6.2, 25.6 M 7.8 / 7.7.  Up to three workers four-wave blocks without runs, then 16 KB held back, in order, as for four.
template <int P>
int launch_quorum_vote(const ss::QuorumVoteArgs &a, hipStream_t stream) {
    const bool few = P <= 2 && a.d < kVoteRuns;
    const size_t block = few ? ss::kBlock : ss::kWave;
    const size_t grid = (a.n_vec + block - 1) / block;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    if constexpr (P <= 2) {
        if (few) return launch(ss::quorum_vote_kernel<P, ss::kBlock, 0, 0, 8>, grid, 0, stream, a);
        return launch(ss::quorum_vote_kernel<P, ss::kWave, 16, 0, 8>, grid, 0, stream, a, ss::kWave);
    } else {
        if constexpr (P == 3) {
            if (a.M == 4 && a.d >= kVoteRuns) return launch(ss::quorum_vote_kernel<P, ss::kWave, 16, 0, 8>, grid, 0, stream, a, ss::kWave);
            if (a.d >= ((size_t)5 << 22) && a.d < kVoteHalves) return launch(ss::quorum_vote_kernel<P, ss::kWave, 0, kVoteChunk, 4>, grid, 0, stream, a, ss::kWave);
        } else {
            if (a.d >= kVoteHalves && a.d < kVoteInOrder) return launch(ss::quorum_vote_kernel<P, ss::kWave, 26, kVoteLongChunk, 8>, grid, 0, stream, a, ss::kWave);
        }
        if (a.d < kVoteHalves) return launch(ss::quorum_vote_kernel<P, ss::kWave, 0, kVoteChunk, 8>, grid, 0, stream, a, ss::kWave);
        return launch(ss::quorum_vote_kernel<P, ss::kWave, 26, 0, 8>, grid, 0, stream, a, ss::kWave);
    }
}

// launch helpers of the ternary (vote with abstention) kernels
template <int BW, int R, int HOLD_KB, bool NEAR, int STORE, uint32_t CHUNK, bool HAS_M, bool VOTE, typename G>
int launch_ternary_shape(ss::TernaryStepArgs &a, size_t d, hipStream_t stream) {
    // the step is one grid over all workers' votes, the pack one row of the grid per worker
    const Tiling t = make_tiling(d, R, true, ss::kWave);
    const size_t grid = t.n_tiles + t.tail_blocks;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    a.n_tiles = (uint32_t)t.n_tiles;
    a.words_total = t.words_total;
    return launch(ss::ternary_step_kernel<BW, R, HOLD_KB, NEAR, STORE, CHUNK, HAS_M, VOTE, G>, grid, 0, stream, a, ss::kWave, VOTE ? 1 : a.M);
}

// The ternary kernel takes any M at run time; its shapes follow the binary step's (launch_step_m, launch_pack_momentum,
// launch_pack_sign).
template <bool HAS_M, bool VOTE, typename G>
int launch_ternary(ss::TernaryStepArgs &a, size_t d, hipStream_t stream) {
    constexpr bool kBf16 = std::is_same<G, ss::Bf16Grad>::value;
    constexpr size_t kBytes = sizeof(typename G::elem) + (HAS_M ? 2 * sizeof(float) : 0);
    using ss::kKeep;
    using ss::kStream;
    using ss::kThrough;
    if constexpr (VOTE) {
        // two rows where a row a lane has too many threads
        if (d >= kOneRowMaxD) return launch_ternary_shape<1, 2, 13, false, kThrough, 0, HAS_M, true, G>(a, d, stream);
        if (a.M == 1 ? one_streams(d, HAS_M) : streams(a.M, d, HAS_M, kBytes)) {
            // us, KB held back: with momentum fp32 11 / 13 / 16: 25.6 M M = 1 80.8 / 84.7 / 92.4, M = 2 125.7 / 133.3 / 146.4, M = 4 217.9 /
            // 219.9 / 235.7, M = 7 367.9 / 360.6 / 375.2, M = 16 868 / 840 / 831, bf16 11 / 12 / 14: M = 3 151.3 / 157.5 / 172.8, M = 8
            // 60 M 840 / 832 / 887; gradients alone 10 / 13: fp32 M = 3 80.2 / 83.1, M = 7 143.2 / 137.6, bf16 M = 7 90.3 / 115.4.
            // One policy for all stores.  A second one for tiles of x that stay in the memory-side cache, as the binary step has, costs these
            // kernels more than it saves.  us, one state again and again / twelve and more in turn, all through / 75 MB of x kept: M = 1
            // gradients alone 60 M 117 / 135 and 117 / 138, bf16 96.5 / 110 and 96.5 / 113, M = 7 25.6 M 142.5 / 145 and 139 / 151, bf16 M = 8 25.6 M 97.4 / 103 and
            // 96.5 / 107, with momentum M = 2 25.6 M 126.7 / 127.7 and 125.8 / 130.7, M = 7 8.0 M 117.8 / 117.9 and 117.6 / 120.9; M = 3 gradients alone 25.6 M 80.3 / 75.8 and
            // 80.6 / 81.3 is the exception.
            // Before (blocks of two to four waves, or eight workers a stage without momentum): M = 2 143, M = 7 387, bf16 60 M 861, fp32
            // gradients M = 7 152.6, bf16 92.4.
            if constexpr (HAS_M) {
                if (a.M < 5) return launch_ternary_shape<1, 1, 11, false, kThrough, 0, true, true, G>(a, d, stream);
                return launch_ternary_shape<1, 1, kBf16 ? 12 : 13, false, kThrough, 0, true, true, G>(a, d, stream);
            } else {
                if (a.M < (kBf16 ? 4 : 5)) return launch_ternary_shape<4, 1, kBf16 ? 7 : 10, false, kThrough, 0, false, true, G>(a, d, stream);
                return launch_ternary_shape<4, 1, kBf16 ? 10 : 13, false, kThrough, 0, false, true, G>(a, d, stream);
            }
        }
        const bool small = d < ((size_t)1 << 20);
        if constexpr (!HAS_M)
            if (a.M == 1 && one_keeps(d, kBf16)) return launch_ternary_shape<8, 1, 0, true, kKeep, 8, false, true, G>(a, d, stream);
        if (small) return launch_ternary_shape<8, 1, 0, true, kStream, 6, HAS_M, true, G>(a, d, stream);
        return launch_ternary_shape<8, 1, 0, true, kStream, 8, HAS_M, true, G>(a, d, stream);
    } else if constexpr (HAS_M) {
        if (d * (size_t)a.M * kBytes < ((size_t)1 << 28)) return launch_ternary_shape<1, 1, 0, false, kStream, 8, true, false, G>(a, d, stream);
        if (d < ((size_t)1 << 25)) return launch_ternary_shape<1, 1, 0, false, kThrough, 9, true, false, G>(a, d, stream);
        return launch_ternary_shape<1, 1, 7, false, kThrough, 0, true, false, G>(a, d, stream);
    } else {
        if (d < ((size_t)1 << 27)) return launch_ternary_shape<1, 2, 0, false, kStream, 8, false, false, G>(a, d, stream);
        return launch_ternary_shape<1, 2, 0, false, kStream, 0, false, false, G>(a, d, stream);
    }
}

template <bool VOTE>
int dispatch_ternary(ss::TernaryStepArgs &a, ss_dtype gdt, bool has_m, size_t d, hipStream_t stream) {
    if (has_m) {
        if (gdt == SS_F32) return launch_ternary<true, VOTE, ss::F32Grad>(a, d, stream);
        return launch_ternary<true, VOTE, ss::Bf16Grad>(a, d, stream);
    }
    if (gdt == SS_F32) return launch_ternary<false, VOTE, ss::F32Grad>(a, d, stream);
    return launch_ternary<false, VOTE, ss::Bf16Grad>(a, d, stream);
}

// answer and update from the planes a pack launch left in a.neg_out / a.zero_out
int launch_quorum_apply(const ss::TernaryStepArgs &t, uint32_t *voted_neg, uint32_t *voted_zero, float *x, size_t d,
                        hipStream_t stream) {
    ss::QuorumApplyArgs a;
    a.neg = t.neg_out;
    a.zero = t.zero_out;
    a.plane_stride = t.plane_stride;
    a.voted_neg = voted_neg;
    a.voted_zero = voted_zero;
    a.x = x;
    a.delta = t.delta;
    a.M = t.M;
    a.quorum = std::min(t.quorum, t.M + 1);   // no quorum above M is ever met: same answers
    a.d = d;
    a.words_total = ss_packed_bytes(d) / 4;
    const bool large = d >= kLargeD;
    const size_t words = large ? 32 : 128;
    const size_t grid = (a.words_total + words - 1) / words;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    const int planes = count_planes(t.M);
    if (planes <= 3)
        return large ? launch(ss::quorum_apply_kernel<3, 8, 1, 0>, grid, 0, stream, a) : launch(ss::quorum_apply_kernel<3, 8, 4, 30>, grid, 0, stream, a);
    if (planes <= 5)
        return large ? launch(ss::quorum_apply_kernel<5, 8, 1, 0>, grid, 0, stream, a) : launch(ss::quorum_apply_kernel<5, 8, 4, 30>, grid, 0, stream, a);
    return large ? launch(ss::quorum_apply_kernel<7, 8, 1, 0>, grid, 0, stream, a) : launch(ss::quorum_apply_kernel<7, 8, 4, 30>, grid, 0, stream, a);
}

}  // namespace

extern "C" {

size_t ss_packed_words(size_t d) { return d / 32 + (d % 32 != 0 ? 1 : 0); }

size_t ss_packed_bytes(size_t d) { return (ss_packed_words(d) * 4 + 15) / 16 * 16; }

int ss_last_hip_error(void) { return g_last_hip_error; }

static int signum_pack_impl(const void *g, ss_dtype gdt, float *m, float beta, uint32_t *packed, size_t d,
                            unsigned flags, void *hip_stream) {
    if (gdt != SS_F32 && gdt != SS_BF16) return SS_ERR_DTYPE;
    if (d == 0) return SS_OK;
    if (!g || !packed) return SS_ERR_NULL;
    if (!aligned16(g) || !aligned16(m) || !aligned16(packed)) return SS_ERR_ALIGN;
    Span spans[3] = {span(g, d * grad_bytes(gdt), false), span(m, d * sizeof(float), true),
                     span(packed, ss_packed_bytes(d), true)};
    if (written_spans_overlap(spans, 3)) return SS_ERR_ARG;
    return launch_pack<1>(1, &g, gdt, m ? &m : nullptr, &packed, beta, flags, d, static_cast<hipStream_t>(hip_stream));
}

int ss_signum_pack(const void *g, ss_dtype gdt, float *m, float beta, uint32_t *packed, size_t d,
                   void *hip_stream) {
    return signum_pack_impl(g, gdt, m, beta, packed, d, SS_STEP_DEFAULT, hip_stream);
}

int ss_signum_pack_warmup(const void *g, ss_dtype gdt, float *m, float beta, uint32_t *packed, size_t d,
                          void *hip_stream) {
    return signum_pack_impl(g, gdt, m, beta, packed, d, SS_STEP_WARMUP, hip_stream);
}

long ss_warmup_length(float beta_f) {
    const double beta = (double)beta_f;
    if (!(beta > 0.0 && beta < 1.0)) return SS_ERR_ARG;
    // smallest C >= 1 with (C/2) beta^C (C+1) (1 - beta^2) <= 1 and beta^(C+1) <= 1/2
    double beta_to_c = 1.0;
    for (long c = 1; c <= SS_WARMUP_MAX; ++c) {
        beta_to_c *= beta;
        const bool bias_settled = 0.5 * (double)c * beta_to_c <= 1.0 / ((1.0 - beta * beta) * ((double)c + 1.0));
        const bool decayed = beta_to_c * beta <= 0.5;
        if (bias_settled && decayed) return c;
    }
    return SS_ERR_RANGE;
}

int ss_majority_vote(const uint32_t *const *packed, int M, uint32_t *voted, size_t d, void *hip_stream) {
    if (M < 1 || M > SS_MAX_WORKERS) return SS_ERR_BAD_M;
    if (d == 0) return SS_OK;
    if (!packed || !voted) return SS_ERR_NULL;
    for (int w = 0; w < M; ++w)
        if (!packed[w]) return SS_ERR_NULL;
    if (!aligned16(voted)) return SS_ERR_ALIGN;
    for (int w = 0; w < M; ++w)
        if (!aligned16(packed[w])) return SS_ERR_ALIGN;
    {
        Span spans[SS_MAX_WORKERS + 1];
        for (int w = 0; w < M; ++w) spans[w] = span(packed[w], ss_packed_bytes(d), false);
        spans[M] = span(voted, ss_packed_bytes(d), true);
        if (written_spans_overlap(spans, M + 1)) return SS_ERR_ARG;
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
#define SS_CASE(n) \
    case n: return launch_vote_fixed<n>(packed, voted, d, stream)
    switch (M) {
        SS_CASE(1); SS_CASE(2); SS_CASE(3); SS_CASE(4); SS_CASE(5); SS_CASE(6); SS_CASE(7); SS_CASE(8);
        SS_CASE(9); SS_CASE(10); SS_CASE(11); SS_CASE(12); SS_CASE(13); SS_CASE(14); SS_CASE(15); SS_CASE(16);
        default: return launch_vote_any(packed, M, voted, d, stream);
    }
#undef SS_CASE
}

int ss_sign_apply(float *x, const uint32_t *bits, float delta, size_t d, void *hip_stream) {
    if (d == 0) return SS_OK;
    if (!x || !bits) return SS_ERR_NULL;
    if (!aligned16(x) || !aligned16(bits)) return SS_ERR_ALIGN;
    Span spans[2] = {span(x, d * sizeof(float), true), span(bits, ss_packed_words(d) * 4, false)};
    if (written_spans_overlap(spans, 2)) return SS_ERR_ARG;
    return launch_apply(ss::apply_kernel<true>, ss::apply_kernel<false>, ss::ApplyArgs{x, bits, delta, 0, d}, hip_stream);
}

// the step over a vector, or a part of one, that every launch shape covers
static int step_part(bool two, const void *const *g, ss_dtype gdt, float *const *m, int M, float beta, float delta, float *x,
                     uint32_t *voted, uint32_t *const *packed, StepVariant var, size_t d, hipStream_t stream) {
    if (two) return launch_two(g, gdt, m, M, beta, delta, x, voted, packed, var, d, stream);
    if (m) {
        if (gdt == SS_F32) return launch_step<true, ss::F32Grad>(M, g, m, packed, beta, delta, x, voted, var, d, stream);
        return launch_step<true, ss::Bf16Grad>(M, g, m, packed, beta, delta, x, voted, var, d, stream);
    }
    if (gdt == SS_F32) return launch_step<false, ss::F32Grad>(M, g, m, packed, beta, delta, x, voted, var, d, stream);
    return launch_step<false, ss::Bf16Grad>(M, g, m, packed, beta, delta, x, voted, var, d, stream);
}

static int vote_step_impl(const void *const *g, ss_dtype gdt, float *const *m, int M, float beta, float delta, float *x,
                          uint32_t *voted, uint32_t *const *packed_out, int8_t *sums_out, size_t d, unsigned flags,
                          void *scratch, size_t scratch_bytes, void *hip_stream) {
    if (M < 1 || M > SS_MAX_WORKERS) return SS_ERR_BAD_M;
    if (gdt != SS_F32 && gdt != SS_BF16) return SS_ERR_DTYPE;
    if (flags & ~(unsigned)(SS_STEP_WARMUP | SS_STEP_SUM_UPDATE)) return SS_ERR_ARG;
    if (d == 0) return SS_OK;
    if (!g || !x || !voted) return SS_ERR_NULL;
    for (int w = 0; w < M; ++w) {
        if (!g[w]) return SS_ERR_NULL;
        if (m && !m[w]) return SS_ERR_NULL;
        if (packed_out && !packed_out[w]) return SS_ERR_NULL;
    }
    if (!aligned16(x) || !aligned16(voted) || !aligned16(sums_out) || !aligned16(scratch)) return SS_ERR_ALIGN;
    for (int w = 0; w < M; ++w) {
        if (!aligned16(g[w])) return SS_ERR_ALIGN;
        if (m && !aligned16(m[w])) return SS_ERR_ALIGN;
        if (packed_out && !aligned16(packed_out[w])) return SS_ERR_ALIGN;
    }
    if (d > kStepMaxD) return SS_ERR_ARG;
    {
        Span spans[3 * SS_MAX_WORKERS + 4];
        int n = 0;
        for (int w = 0; w < M; ++w) {
            spans[n++] = span(g[w], d * grad_bytes(gdt), false);
            if (m) spans[n++] = span(m[w], d * sizeof(float), true);
            if (packed_out) spans[n++] = span(packed_out[w], ss_packed_bytes(d), true);
        }
        spans[n++] = span(x, d * sizeof(float), true);
        spans[n++] = span(voted, ss_packed_bytes(d), true);
        spans[n++] = span(sums_out, d, true);
        spans[n++] = span(scratch, scratch_bytes, true);
        if (written_spans_overlap(spans, n)) return SS_ERR_ARG;
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    // Two launches that hand the signs over through the caller's bit buffers, or through the lent memory over as much
    // of the vector at a time as it has room for; otherwise one pass.  Same results, bit for bit.
    const size_t slab = scratch && !packed_out ? scratch_slab(M, d, scratch_bytes) : 0;
    const bool lent = slab >= kScratchMinSlab;
    const bool two = lent || (packed_out && split_pays(M, d, m != nullptr, grad_bytes(gdt) + (m ? 2 * sizeof(float) : 0)));
    const size_t part = lent ? slab : std::min(d, kOneRowMaxD);
    if (!lent && part == d)
        return step_part(two, g, gdt, m, M, beta, delta, x, voted, packed_out, StepVariant{flags, sums_out}, d, stream);
    const size_t stride = ss_packed_bytes(part);
    for (size_t lo = 0; lo < d; lo += part) {
        const void *gs[SS_MAX_WORKERS];
        float *ms[SS_MAX_WORKERS];
        uint32_t *ps[SS_MAX_WORKERS];
        for (int w = 0; w < M; ++w) {
            gs[w] = static_cast<const char *>(g[w]) + lo * grad_bytes(gdt);
            ms[w] = m ? m[w] + lo : nullptr;
            if (lent) ps[w] = reinterpret_cast<uint32_t *>(static_cast<char *>(scratch) + w * stride);
            else ps[w] = packed_out ? packed_out[w] + lo / 32 : nullptr;
        }
        const int rc = step_part(two, gs, gdt, m ? ms : nullptr, M, beta, delta, x + lo, voted + lo / 32,
                                 lent || packed_out ? ps : nullptr, StepVariant{flags, sums_out ? sums_out + lo : nullptr},
                                 std::min(part, d - lo), stream);
        if (rc != SS_OK) return rc;
    }
    return SS_OK;
}

int ss_signum_vote_step_ex(const void *const *g, ss_dtype gdt, float *const *m, int M, float beta, float delta,
                           float *x, uint32_t *voted, uint32_t *const *packed_out, int8_t *sums_out, size_t d,
                           unsigned flags, void *hip_stream) {
    return vote_step_impl(g, gdt, m, M, beta, delta, x, voted, packed_out, sums_out, d, flags, nullptr, 0, hip_stream);
}

size_t ss_step_scratch_bytes(ss_dtype gdt, int has_momentum, int M, size_t d) {
    if (M < 2 || M > SS_MAX_WORKERS || (gdt != SS_F32 && gdt != SS_BF16) || !has_momentum) return 0;
    if (d < kScratchMinSlab || !scratch_pays(M, d, grad_bytes(gdt) + sizeof(float) * 2)) return 0;
    return (size_t)M * ss_packed_bytes(scratch_slab(M, d, kScratchBytes));
}

int ss_signum_vote_step_scratch(const void *const *g, ss_dtype gdt, float *const *m, int M, float beta, float delta,
                                float *x, uint32_t *voted, int8_t *sums_out, void *scratch, size_t scratch_bytes,
                                size_t d, unsigned flags, void *hip_stream) {
    return vote_step_impl(g, gdt, m, M, beta, delta, x, voted, nullptr, sums_out, d, flags, scratch,
                          scratch ? scratch_bytes : 0, hip_stream);
}

int ss_signum_vote_step(const void *const *g, ss_dtype gdt, float *const *m, int M, float beta, float delta,
                        float *x, uint32_t *voted, uint32_t *const *packed_out, size_t d, void *hip_stream) {
    return ss_signum_vote_step_ex(g, gdt, m, M, beta, delta, x, voted, packed_out, nullptr, d, SS_STEP_DEFAULT,
                                  hip_stream);
}

int ss_vote_sum(const uint32_t *const *packed, int M, int8_t *sums, size_t d, void *hip_stream) {
    if (M < 1 || M > SS_MAX_WORKERS) return SS_ERR_BAD_M;
    if (d == 0) return SS_OK;
    if (!packed || !sums) return SS_ERR_NULL;
    for (int w = 0; w < M; ++w)
        if (!packed[w]) return SS_ERR_NULL;
    if (!aligned16(sums)) return SS_ERR_ALIGN;
    for (int w = 0; w < M; ++w)
        if (!aligned16(packed[w])) return SS_ERR_ALIGN;
    {
        Span spans[SS_MAX_WORKERS + 1];
        for (int w = 0; w < M; ++w) spans[w] = span(packed[w], ss_packed_bytes(d), false);
        spans[M] = span(sums, d, true);
        if (written_spans_overlap(spans, M + 1)) return SS_ERR_ARG;
    }
    ss::VoteSumArgs a;
    for (int w = 0; w < SS_MAX_WORKERS; ++w) a.packed[w] = w < M ? packed[w] : nullptr;
    a.sums = sums;
    a.M = M;
    a.d = d;
    a.n_vec = ss_packed_bytes(d) / 16;
    const size_t grid = (a.n_vec + ss::kWave - 1) / ss::kWave;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (sum_word_lanes(M, d)) {
        const size_t blocks = (4 * a.n_vec + 63) / 64;
        const int planes = count_planes(M);
        if (planes <= 3) return launch(ss::vote_sum_word_kernel<3>, blocks, 0, stream, a, 64);
        if (planes <= 5) return launch(ss::vote_sum_word_kernel<5>, blocks, 0, stream, a, 64);
        return launch(ss::vote_sum_word_kernel<7>, blocks, 0, stream, a, 64);
    }
    switch (count_planes(M)) {
        case 1: return launch_vote_sum<1>(a, grid, stream);
        case 2: return launch_vote_sum<2>(a, grid, stream);
        case 3: return launch_vote_sum<3>(a, grid, stream);
        case 4: return launch_vote_sum<4>(a, grid, stream);
        case 5: return launch_vote_sum<5>(a, grid, stream);
        case 6: return launch_vote_sum<6>(a, grid, stream);
        default: return launch_vote_sum<7>(a, grid, stream);
    }
}

int ss_sum_apply(float *x, const int8_t *sums, float delta, size_t d, void *hip_stream) {
    if (d == 0) return SS_OK;
    if (!x || !sums) return SS_ERR_NULL;
    if (!aligned16(x) || !aligned16(sums)) return SS_ERR_ALIGN;
    Span spans[2] = {span(x, d * sizeof(float), true), span(sums, d, false)};
    if (written_spans_overlap(spans, 2)) return SS_ERR_ARG;
    return launch_apply(ss::sum_apply_kernel<true>, ss::sum_apply_kernel<false>, ss::SumApplyArgs{x, sums, delta, 0, d}, hip_stream);
}

int ss_welford_update(const void *g, ss_dtype gdt, float *mean, float *m2, uint64_t n, size_t d, void *hip_stream) {
    if (gdt != SS_F32 && gdt != SS_BF16) return SS_ERR_DTYPE;
    if (n < 1 || n > (1ull << 24)) return SS_ERR_ARG;   // n must be exact in fp32
    if (d == 0) return SS_OK;
    if (!g || !mean || !m2) return SS_ERR_NULL;
    if (!aligned16(g) || !aligned16(mean) || !aligned16(m2)) return SS_ERR_ALIGN;
    Span spans[3] = {span(g, d * grad_bytes(gdt), false), span(mean, d * sizeof(float), true),
                     span(m2, d * sizeof(float), true)};
    if (written_spans_overlap(spans, 3)) return SS_ERR_ARG;
    const Tiling t = make_tiling(d, 1, false, ss::kWave);
    const size_t grid = t.n_tiles + t.tail_blocks;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    const ss::WelfordArgs a{g, mean, m2, (float)n, (uint32_t)t.n_tiles, d};
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    // From 2^21 coordinates on m2 is left in the memory-side cache (kKeep) for the next update and for sigma, the mean as long as both are not
    // too much for it: runs of half a megabyte a die below 2^24, in order with 14 waves a unit beyond.  us, update, sigma and two densities,
    // everything written through / m2 and sigma kept / the mean too, in order: 8.8 M 61.6 / 57.4 / 56.5
    // (runs 55.7), 17.6 M 105.8 / 99.3 / 98.2 (runs 100.5), 30 M 169.2 / 158.1 / 156.9, 40 M 220.0 / 205.1 / 205.5, 48 M 261.6 / 243.8 / 251.0, 60 M 323 / 302 / 317, 138 M
    // 742 / 736 / 742; m2 alone kept 60 M 303.6, 80 M 405.5 (428, with sigma 419.7), 138 M 715, 390 M 2,024 (2,059).
    // An update that nothing reads soon gains nothing: twelve states and more in turn, and one behind a 600 MB copy (copy and update), to the L2 or through / so: 4.4 M 15.4 / 16.3 and 127.4 /
    // 128.0, 8.8 M 28.5 / 29.5 and 142.0 / 142.3, 25.6 M 78.0 / 78.1 and 189.0 / 193.2, 40 M 118.9 / 119.6 and 229.9 / 237.9, 138 M 409.1 / 408.9 and 529.7 / 527.5.  Below 2^21 it
    // loses and the four calls together gain little: kept in order against runs to the L2, twelve and more in turn, update alone 272,474 2.76 / 2.53, 700,001 4.44 / 3.56, 1.1 M 6.27 / 5.04,
    // 1.8 M 8.32 / 7.43, all four 12.25 / 12.58, 15.83 / 15.88, 17.3 / 18.0, 21.2 / 22.4.
    using ss::kKeep;
    using ss::kStream;
    using ss::kThrough;
    const bool small = d < ((size_t)1 << 21), runs = d < ((size_t)1 << 24), both = d < ((size_t)5 << 23);
    if (gdt == SS_F32) {
        if (small) return launch(ss::welford_update_kernel<0, kStream, kStream, 9, ss::F32Grad>, grid, 0, stream, a, ss::kWave);
        if (runs) return launch(ss::welford_update_kernel<0, kKeep, kKeep, 9, ss::F32Grad>, grid, 0, stream, a, ss::kWave);
        if (both) return launch(ss::welford_update_kernel<11, kKeep, kKeep, 0, ss::F32Grad>, grid, 0, stream, a, ss::kWave);
        return launch(ss::welford_update_kernel<11, kThrough, kKeep, 0, ss::F32Grad>, grid, 0, stream, a, ss::kWave);
    }
    if (small) return launch(ss::welford_update_kernel<0, kStream, kStream, 9, ss::Bf16Grad>, grid, 0, stream, a, ss::kWave);
    if (runs) return launch(ss::welford_update_kernel<0, kKeep, kKeep, 9, ss::Bf16Grad>, grid, 0, stream, a, ss::kWave);
    if (both) return launch(ss::welford_update_kernel<11, kKeep, kKeep, 0, ss::Bf16Grad>, grid, 0, stream, a, ss::kWave);
    return launch(ss::welford_update_kernel<11, kThrough, kKeep, 0, ss::Bf16Grad>, grid, 0, stream, a, ss::kWave);
}

int ss_welford_sigma(const float *m2, uint64_t n, float *sigma, size_t d, void *hip_stream) {
    if (n < 1 || n > (1ull << 24)) return SS_ERR_ARG;
    if (d == 0) return SS_OK;
    if (!m2 || !sigma) return SS_ERR_NULL;
    if (!aligned16(m2) || !aligned16(sigma)) return SS_ERR_ALIGN;
    Span spans[2] = {span(m2, d * sizeof(float), false), span(sigma, d * sizeof(float), true)};
    if (written_spans_overlap(spans, 2)) return SS_ERR_ARG;
    const bool two_rows = d >= kOneRowMaxD;
    const Tiling t = make_tiling(d, two_rows ? 2 : 1, false, ss::kWave);
    const size_t grid = t.n_tiles + t.tail_blocks;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    const ss::SigmaArgs a{m2, sigma, (float)n, (uint32_t)t.n_tiles, d};
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (two_rows) return launch(ss::welford_sigma_kernel<2, ss::kThrough>, grid, 0, stream, a, ss::kWave);
    // kept for the density that reads it next while the cache can hold all of it: 60 M 301.8 us of statistics against 303.6, 80 M 419.7 / 405.5.
    // By itself over sixty vectors in turn, to the L2 or through / kept: 272,474 2.34 / 2.49, 1.1 M 3.24 / 3.6, 4.4 M 7.6 / 7.8, 25.6 M 31.9 / 32.1.
    if (d >= ((size_t)1 << 26)) return launch(ss::welford_sigma_kernel<1, ss::kThrough>, grid, 0, stream, a, ss::kWave);
    return launch(ss::welford_sigma_kernel<1, ss::kKeep>, grid, 0, stream, a, ss::kWave);
}

size_t ss_density_workspace_bytes(void) { return sizeof(ss::DensityScratch); }

// Rows of a density tile: short tiles while the blocks are few, eight rows where their number, that is the tickets', counts, and six,
// whose 48 KB do not line blocks up on the same channels, where memory decides.  us, 3 / 8 / 6 rows: 100,003 3.7 / 3.8 / 3.8, 272,474 4.15 / 4.8 / 4.6,
// 700,001 4.9 / 5.0 / 4.8, 1.1 M 5.8 / 5.0 / 5.0, 4.4 M 8.2 / 7.3 / 7.6, 25.6 M 19.0 / 18.7 / 19.1, 60 M 37.2 / 37.8 / 37.1, 100 M 59.1 / 64.3 / 58.7, 390 M
// 217 / 226 / 217; four 86.6 at 138 M, two of which the next two are loaded early 80.8, six 79.7.
static int density_rows(size_t d) { return d < ((size_t)3 << 18) ? 3 : d < ((size_t)1 << 25) ? 8 : 6; }

// `partials` is a device address: the caller's workspace, or the looked-up address of the array above
static int density_impl(const float *v, size_t d, double *out, ss::DensityScratch *partials, hipStream_t stream) {
    ss::DensityArgs a;
    a.v = v;
    a.out = out;
    a.scratch = partials;
    a.d = d;
    a.n_rows = d / ((size_t)ss::kDensityThreads * ss::kQuad);
    const int rows = density_rows(d);
    a.n_tiles = a.n_rows / rows;
    // every block gets the same number of tiles (the last one possibly fewer): the grid is a
    // function of d alone, which is what fixes the order of the additions
    const size_t per_block = (a.n_tiles + ss::kDensityMaxBlocks - 1) / ss::kDensityMaxBlocks;
    const size_t grid = per_block ? (a.n_tiles + per_block - 1) / per_block : 1;
    if (rows == 3) return launch(ss::density_kernel<3>, grid, 0, stream, a, ss::kDensityThreads);
    if (rows == 6) return launch(ss::density_kernel<6>, grid, 0, stream, a, ss::kDensityThreads);
    return launch(ss::density_kernel<8>, grid, 0, stream, a, ss::kDensityThreads);
}

int ss_density(const float *v, size_t d, double *out, void *workspace, void *hip_stream) {
    if (!out || !workspace) return SS_ERR_NULL;
    if (d > 0 && !v) return SS_ERR_NULL;
    if (!aligned16(v) || !aligned16(out) || !aligned16(workspace)) return SS_ERR_ALIGN;
    Span spans[3] = {span(out, 3 * sizeof(double), true), span(workspace, sizeof(ss::DensityScratch), true),
                     span(v, d * sizeof(float), false)};
    if (written_spans_overlap(spans, 3)) return SS_ERR_ARG;
    return density_impl(v, d, out, static_cast<ss::DensityScratch *>(workspace), static_cast<hipStream_t>(hip_stream));
}

int ss_density_static(const float *v, size_t d, double *out, void *hip_stream) {
    if (!out) return SS_ERR_NULL;
    if (d > 0 && !v) return SS_ERR_NULL;
    if (!aligned16(v) || !aligned16(out)) return SS_ERR_ALIGN;
    if (d > SS_DENSITY_STATIC_MAX_D) return SS_ERR_RANGE;
    Span spans[2] = {span(out, 3 * sizeof(double), true), span(v, d * sizeof(float), false)};
    if (written_spans_overlap(spans, 2)) return SS_ERR_ARG;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        return SS_ERR_HIP;
    }
    if (dev < 0 || dev >= kMaxDevices) return SS_ERR_ARG;
    ss::DensityScratch *on_device = g_scratch_on_device[dev].load(std::memory_order_acquire);
    if (!on_device) {
        // first call on this device (which is current): every device holds its own copy of the
        // array at its own address.  Two threads racing here look up the same address.
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            g_last_hip_error = (int)e;
            return SS_ERR_HIP;
        }
        on_device = static_cast<ss::DensityScratch *>(p);
        g_scratch_on_device[dev].store(on_device, std::memory_order_release);
    }
    return density_impl(v, d, out, on_device, static_cast<hipStream_t>(hip_stream));
}

// ---- majority vote with abstention ----

int ss_signum_pack_ternary(const void *g, ss_dtype gdt, float *m, float beta, float tau, uint32_t *neg,
                           uint32_t *zero, size_t d, void *hip_stream) {
    if (gdt != SS_F32 && gdt != SS_BF16) return SS_ERR_DTYPE;
    if (!(tau >= 0.0f)) return SS_ERR_ARG;
    if (d == 0) return SS_OK;
    if (!g || !neg || !zero) return SS_ERR_NULL;
    if (!aligned16(g) || !aligned16(m) || !aligned16(neg) || !aligned16(zero)) return SS_ERR_ALIGN;
    Span spans[4] = {span(g, d * grad_bytes(gdt), false), span(m, d * sizeof(float), true),
                     span(neg, ss_packed_bytes(d), true), span(zero, ss_packed_bytes(d), true)};
    if (written_spans_overlap(spans, 4)) return SS_ERR_ARG;
    ss::TernaryStepArgs a{};
    a.g[0] = g;
    a.m[0] = m;
    a.neg_out = neg;
    a.zero_out = zero;
    a.beta = beta;
    a.omb = 1.0f - beta;
    a.tau = tau;
    a.M = 1;
    a.quorum = 1;
    a.d = d;
    return dispatch_ternary<false>(a, gdt, m != nullptr, d, static_cast<hipStream_t>(hip_stream));
}

int ss_quorum_vote(const uint32_t *const *neg, const uint32_t *const *zero, int M, int quorum,
                   uint32_t *voted_neg, uint32_t *voted_zero, size_t d, void *hip_stream) {
    if (M < 1 || M > SS_MAX_WORKERS) return SS_ERR_BAD_M;
    if (quorum < 1) return SS_ERR_ARG;
    if (d == 0) return SS_OK;
    if (!neg || !zero || !voted_neg || !voted_zero) return SS_ERR_NULL;
    for (int w = 0; w < M; ++w)
        if (!neg[w] || !zero[w]) return SS_ERR_NULL;
    if (!aligned16(voted_neg) || !aligned16(voted_zero)) return SS_ERR_ALIGN;
    for (int w = 0; w < M; ++w)
        if (!aligned16(neg[w]) || !aligned16(zero[w])) return SS_ERR_ALIGN;
    {
        Span spans[2 * SS_MAX_WORKERS + 2];
        for (int w = 0; w < M; ++w) {
            spans[2 * w] = span(neg[w], ss_packed_bytes(d), false);
            spans[2 * w + 1] = span(zero[w], ss_packed_bytes(d), false);
        }
        spans[2 * M] = span(voted_neg, ss_packed_bytes(d), true);
        spans[2 * M + 1] = span(voted_zero, ss_packed_bytes(d), true);
        if (written_spans_overlap(spans, 2 * M + 2)) return SS_ERR_ARG;
    }
    ss::QuorumVoteArgs a{};
    for (int w = 0; w < M; ++w) {
        a.neg[w] = neg[w];
        a.zero[w] = zero[w];
    }
    a.voted_neg = voted_neg;
    a.voted_zero = voted_zero;
    a.M = M;
    a.quorum = quorum > M + 1 ? M + 1 : quorum;   // any quorum above M can never be met: same answers
    a.d = d;
    a.n_vec = ss_packed_bytes(d) / 16;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (sum_word_lanes(M, d)) {
        const size_t blocks = (4 * a.n_vec + 63) / 64;
        const int planes = count_planes(M);
        if (planes <= 3) return launch(ss::quorum_word_kernel<3>, blocks, 0, stream, a, 64);
        if (planes <= 5) return launch(ss::quorum_word_kernel<5>, blocks, 0, stream, a, 64);
        return launch(ss::quorum_word_kernel<7>, blocks, 0, stream, a, 64);
    }
    switch (count_planes(M)) {
        case 1: return launch_quorum_vote<1>(a, stream);
        case 2: return launch_quorum_vote<2>(a, stream);
        case 3: return launch_quorum_vote<3>(a, stream);
        case 4: return launch_quorum_vote<4>(a, stream);
        case 5: return launch_quorum_vote<5>(a, stream);
        case 6: return launch_quorum_vote<6>(a, stream);
        default: return launch_quorum_vote<7>(a, stream);
    }
}

int ss_ternary_apply(float *x, const uint32_t *neg, const uint32_t *zero, float delta, size_t d,
                     void *hip_stream) {
    if (d == 0) return SS_OK;
    if (!x || !neg || !zero) return SS_ERR_NULL;
    if (!aligned16(x) || !aligned16(neg) || !aligned16(zero)) return SS_ERR_ALIGN;
    Span spans[3] = {span(x, d * sizeof(float), true), span(neg, ss_packed_words(d) * 4, false),
                     span(zero, ss_packed_words(d) * 4, false)};
    if (written_spans_overlap(spans, 3)) return SS_ERR_ARG;
    return launch_apply(ss::ternary_apply_kernel<true>, ss::ternary_apply_kernel<false>,
                        ss::TernaryApplyArgs{x, neg, zero, delta, 0, d}, hip_stream);
}

static int ternary_step_impl(const void *const *g, ss_dtype gdt, float *const *m, int M, float beta, float tau, int quorum,
                             float delta, float *x, uint32_t *voted_neg, uint32_t *voted_zero, void *scratch,
                             size_t scratch_bytes, size_t d, void *hip_stream) {
    if (M < 1 || M > SS_MAX_WORKERS) return SS_ERR_BAD_M;
    if (gdt != SS_F32 && gdt != SS_BF16) return SS_ERR_DTYPE;
    if (!(tau >= 0.0f) || quorum < 1) return SS_ERR_ARG;
    if (d == 0) return SS_OK;
    if (!g || !x || !voted_neg || !voted_zero) return SS_ERR_NULL;
    for (int w = 0; w < M; ++w) {
        if (!g[w]) return SS_ERR_NULL;
        if (m && !m[w]) return SS_ERR_NULL;
    }
    if (!aligned16(x) || !aligned16(voted_neg) || !aligned16(voted_zero) || !aligned16(scratch)) return SS_ERR_ALIGN;
    for (int w = 0; w < M; ++w) {
        if (!aligned16(g[w])) return SS_ERR_ALIGN;
        if (m && !aligned16(m[w])) return SS_ERR_ALIGN;
    }
    {
        Span spans[2 * SS_MAX_WORKERS + 4];
        int n = 0;
        for (int w = 0; w < M; ++w) {
            spans[n++] = span(g[w], d * grad_bytes(gdt), false);
            if (m) spans[n++] = span(m[w], d * sizeof(float), true);
        }
        spans[n++] = span(x, d * sizeof(float), true);
        spans[n++] = span(voted_neg, ss_packed_bytes(d), true);
        spans[n++] = span(voted_zero, ss_packed_bytes(d), true);
        spans[n++] = span(scratch, scratch_bytes, true);
        if (written_spans_overlap(spans, n)) return SS_ERR_ARG;
    }
    ss::TernaryStepArgs a{};
    for (int w = 0; w < M; ++w) {
        a.g[w] = g[w];
        a.m[w] = m ? m[w] : nullptr;
    }
    a.x = x;
    a.voted_neg = voted_neg;
    a.voted_zero = voted_zero;
    a.beta = beta;
    a.omb = 1.0f - beta;
    a.delta = delta;
    a.tau = tau;
    a.M = M;
    a.quorum = quorum;
    a.d = d;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const size_t slab = scratch ? scratch_slab(2 * M, d, scratch_bytes) : 0;
    if (slab < kScratchMinSlab) return dispatch_ternary<true>(a, gdt, m != nullptr, d, stream);
    // pack over all workers, then answer and update, over as much of the vector as the lent memory holds
    const size_t plane = ss_packed_bytes(slab) / 4;
    a.neg_out = static_cast<uint32_t *>(scratch);
    a.zero_out = a.neg_out + plane;
    a.plane_stride = 2 * plane;
    for (size_t lo = 0; lo < d; lo += slab) {
        const size_t n = std::min(slab, d - lo);
        for (int w = 0; w < M; ++w) {
            a.g[w] = static_cast<const char *>(g[w]) + lo * grad_bytes(gdt);
            a.m[w] = m ? m[w] + lo : nullptr;
        }
        a.d = n;
        int rc = dispatch_ternary<false>(a, gdt, m != nullptr, n, stream);
        if (rc == SS_OK) rc = launch_quorum_apply(a, voted_neg + lo / 32, voted_zero + lo / 32, x + lo, n, stream);
        if (rc != SS_OK) return rc;
    }
    return SS_OK;
}

int ss_signum_vote_step_ternary(const void *const *g, ss_dtype gdt, float *const *m, int M, float beta, float tau,
                                int quorum, float delta, float *x, uint32_t *voted_neg, uint32_t *voted_zero,
                                size_t d, void *hip_stream) {
    return ternary_step_impl(g, gdt, m, M, beta, tau, quorum, delta, x, voted_neg, voted_zero, nullptr, 0, d, hip_stream);
}

size_t ss_ternary_scratch_bytes(ss_dtype gdt, int has_momentum, int M, size_t d) {
    if (ss_step_scratch_bytes(gdt, has_momentum, M, d) == 0) return 0;
    return (size_t)(2 * M) * ss_packed_bytes(scratch_slab(2 * M, d, kScratchBytes));
}

int ss_signum_vote_step_ternary_scratch(const void *const *g, ss_dtype gdt, float *const *m, int M, float beta,
                                        float tau, int quorum, float delta, float *x, uint32_t *voted_neg,
                                        uint32_t *voted_zero, void *scratch, size_t scratch_bytes, size_t d,
                                        void *hip_stream) {
    return ternary_step_impl(g, gdt, m, M, beta, tau, quorum, delta, x, voted_neg, voted_zero, scratch,
                             scratch ? scratch_bytes : 0, d, hip_stream);
}


int ss_stream_copy(void *dst, const void *src, size_t nbytes, void *hip_stream) {
    if (nbytes == 0) return SS_OK;
    if (!dst || !src) return SS_ERR_NULL;
    if (!aligned16(dst) || !aligned16(src)) return SS_ERR_ALIGN;
    if (nbytes % 16 != 0) return SS_ERR_ARG;
    Span spans[2] = {span(dst, nbytes, true), span(src, nbytes, false)};
    if (written_spans_overlap(spans, 2)) return SS_ERR_ARG;
    const size_t n_vec = nbytes / 16;
    const size_t grid = (n_vec + ss::kWave - 1) / ss::kWave;
    if (grid > kMaxGrid) return SS_ERR_ARG;
    const ss::CopyArgs a{static_cast<ss::f32x4 *>(dst), static_cast<const ss::f32x4 *>(src), n_vec};
    return launch(ss::copy_kernel, grid, 0, static_cast<hipStream_t>(hip_stream), a, ss::kWave);
}

}  // extern "C"
