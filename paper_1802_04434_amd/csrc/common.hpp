// Shared device helpers for the gfx950 kernels of the signSGD / Signum
// majority-vote step (arxiv 1802.04434, Algorithms 1-3).
//
// Geometry used by every streaming kernel here
//   lane      owns 4 consecutive coordinates ("quad" q = coordinates 4q..4q+3):
//             one 128-bit access per fp32 buffer, one 64-bit access for bf16
//   8 lanes   own 32 consecutive coordinates = one packed word
//   wave      64 lanes = 256 coordinates = 8 packed words
//   block     one wave (kWave) with one row of 256 coordinates or a few; B threads = 4 B coordinates
//             per row where a kernel is launched with more
// The coordinates that do not fill a whole tile go through a scalar path in
// extra blocks at the end of the same grid (one coordinate per lane; there a
// wave ballot is already in packed-word order).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#pragma clang fp contract(off)

namespace ss {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;            // threads of the one-wave blocks
constexpr int kBlock = 256;          // threads of the four-wave blocks
constexpr int kQuad = 4;             // coordinates per lane per row
constexpr int kRowCoords = kBlock * kQuad;   // 1024

// Streaming accesses: every byte is touched once per step, so mark them
// non-temporal and keep them out of the way of anything cached.
template <typename T>
__device__ __forceinline__ T ld_stream(const T *p) {
    return __builtin_nontemporal_load(p);
}
template <typename T>
__device__ __forceinline__ void st_stream(T *p, T v) {
    __builtin_nontemporal_store(v, p);
}

// A block's own part of a buffer as a buffer descriptor: the base is the same for the whole block and sits in
// scalar registers, a lane adds a 32-bit byte offset.  What lies at or beyond `bytes` reads as zero and is
// not written.  Kernels that write where they have read are 1-2 % faster with it than with a 64-bit address a lane
// (pack of 138 M coordinates, M = 4 968 us against 979, 400 M, M = 2 1,437 / 1,464); kernels that only read are as much slower
// (a wave lives for ~2 us and the descriptors lengthen its start) and keep addresses.
typedef __amdgpu_buffer_rsrc_t Window;
__device__ __forceinline__ Window window(const void *base, size_t from, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(static_cast<const char *>(base)) + from, 0, (int)bytes, 0x00020000);
}

// Cache policies of stores (bits of the instruction: 2 = nt, 16 = sc1).  kStream leaves a written line to the L2 to write back,
// kThrough sends it on at once; nt also keeps it out of the 256 MB memory-side cache.  kKeep sends it on and leaves it there, for
// the next step or kernel that reads it.  Updating a vector in place (nt loads, which find what is there and do not crowd it out),
// us, kStream / kThrough / kKeep: the same 4.4 M coordinates again 6.8 / 7.0 / 6.2, 25.6 M 31.3 / 31.0 / 28.4, 60 M (240 MB) 72.0 / 70.4 / 65.0; too much for
// the cache, twelve vectors of 8.8 M in turn 12.1 / 11.9 / 12.2, of 138 M 163.4 / 161.5 / 164.3.
constexpr int kStream = 2, kKeep = 16, kThrough = 18;

__device__ __forceinline__ f32x4 ld_quad(Window w, uint32_t off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(w, (int)off, 0, kStream));
}
template <int STORE>
__device__ __forceinline__ void st_quad(Window w, uint32_t off, f32x4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), w, (int)off, 0, STORE);
}

// A tile's quad at byte offset `off`, through a descriptor, or - NEAR, for buffers of less than 4 GiB - at a 32-bit
// offset from the buffer's own base, which costs the wave no arithmetic per buffer: launches of a few
// microseconds are as long as their waves' first instructions take.
template <bool NEAR>
__device__ __forceinline__ f32x4 ld_tile(const void *base, size_t tile, uint32_t tile_bytes, uint32_t off) {
    if constexpr (NEAR)
        return ld_stream(reinterpret_cast<const f32x4 *>(static_cast<const char *>(base) + (uint32_t)((uint32_t)tile * tile_bytes + off)));
    else return ld_quad(window(base, tile * tile_bytes, tile_bytes), off);
}
template <bool NEAR, int STORE>
__device__ __forceinline__ void st_tile(float *base, size_t tile, uint32_t tile_bytes, uint32_t off, f32x4 v) {
    if constexpr (!NEAR) st_quad<STORE>(window(base, tile * tile_bytes, tile_bytes), off, v);
    // addresses know nt: the other policies take a descriptor of the whole buffer, made while the loads are out
    else if constexpr (STORE != kStream) st_quad<STORE>(window(base, 0, 0xFFFFFFFFu), (uint32_t)tile * tile_bytes + off, v);
    else st_stream(reinterpret_cast<f32x4 *>(reinterpret_cast<char *>(base) + (uint32_t)((uint32_t)tile * tile_bytes + off)), v);
}

// bf16 -> fp32 is exact: the bf16 pattern is the upper half of the fp32
__device__ __forceinline__ float widen_bf16(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

struct F32Grad {
    typedef float elem;
    static __device__ __forceinline__ f32x4 load4(const void *base, size_t quad) {
        return ld_stream(reinterpret_cast<const f32x4 *>(base) + quad);
    }
    static __device__ __forceinline__ f32x4 load4(Window w, uint32_t quad) { return ld_quad(w, quad * 16); }
    template <bool NEAR>
    static __device__ __forceinline__ f32x4 load_tile(const void *base, size_t tile, uint32_t tile_bytes, uint32_t quad) {
        return ld_tile<NEAR>(base, tile, tile_bytes, quad * 16);
    }
    static __device__ __forceinline__ float load1(const void *base, size_t i) {
        return reinterpret_cast<const float *>(base)[i];
    }
};

struct Bf16Grad {
    typedef uint16_t elem;
    static __device__ __forceinline__ f32x4 widen(u16x4 r) {
        f32x4 o;
        o.x = widen_bf16(r.x); o.y = widen_bf16(r.y); o.z = widen_bf16(r.z); o.w = widen_bf16(r.w);
        return o;
    }
    static __device__ __forceinline__ f32x4 load4(const void *base, size_t quad) {
        return widen(ld_stream(reinterpret_cast<const u16x4 *>(base) + quad));
    }
    static __device__ __forceinline__ f32x4 load4(Window w, uint32_t quad) {
        return widen(__builtin_bit_cast(u16x4, __builtin_amdgcn_raw_buffer_load_b64(w, (int)(quad * 8), 0, kStream)));
    }
    template <bool NEAR>
    static __device__ __forceinline__ f32x4 load_tile(const void *base, size_t tile, uint32_t tile_bytes, uint32_t quad) {
        if constexpr (NEAR)
            return widen(ld_stream(reinterpret_cast<const u16x4 *>(static_cast<const char *>(base) + (uint32_t)((uint32_t)tile * tile_bytes + quad * 8))));
        else return load4(window(base, tile * tile_bytes, tile_bytes), quad);
    }
    static __device__ __forceinline__ float load1(const void *base, size_t i) {
        return widen_bf16(reinterpret_cast<const uint16_t *>(base)[i]);
    }
};

// Algorithm 2's momentum line in fp32 with three roundings (two products, one
// sum); the file is compiled with contraction off so no FMA is formed.
__device__ __forceinline__ float momentum(float beta, float omb, float m, float g) {
    float t1 = beta * m;
    float t2 = omb * g;
    return t1 + t2;
}

// sign(v) = -1 exactly when v < 0 (zeros of either sign and NaN are "+")
__device__ __forceinline__ uint32_t neg_bit(float v) { return v < 0.0f ? 1u : 0u; }

__device__ __forceinline__ uint32_t neg_nibble(f32x4 v) {
    return neg_bit(v.x) | (neg_bit(v.y) << 1) | (neg_bit(v.z) << 2) | (neg_bit(v.w) << 3);
}

// signs of eight bf16, the lower coordinate in the lower half of a word
__device__ __forceinline__ uint32_t neg_byte_bf16(u32x4 v) {
    uint32_t byte = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        byte |= neg_bit(widen_bf16((uint16_t)v[k])) << (2 * k);
        byte |= neg_bit(widen_bf16((uint16_t)(v[k] >> 16))) << (2 * k + 1);
    }
    return byte;
}

// Algorithm 3's worker update for one coordinate: s = -1 where `neg`
__device__ __forceinline__ float step(float x, float delta, bool neg) {
    return neg ? x + delta : x - delta;
}

// OR-combine the 4-bit sign nibbles of 8 neighbouring lanes (lane & 7 = 0..7)
// into the 32-bit packed word of their 32 coordinates; every one of the 8
// lanes ends up holding the word.  Three DPP moves inside a row of 16 lanes:
// swap lanes within pairs, swap pairs within a quad, then mirror each group of
// 8 (lane i <-> 7-i), which after the first two steps brings in the other
// quad's value whichever lane it comes from.
__device__ __forceinline__ uint32_t combine8(uint32_t nibble, int lane) {
    uint32_t v = nibble << ((lane & 7) * 4);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1 /* quad_perm [1,0,3,2] */, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E /* quad_perm [2,3,0,1] */, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141 /* row_half_mirror */, 0xF, 0xF, false);
    return v;
}

// the same for a byte of signs (8 coordinates) in each of 4 neighbouring lanes
__device__ __forceinline__ uint32_t combine4(uint32_t byte, int lane) {
    uint32_t v = byte << ((lane & 3) * 8);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1 /* quad_perm [1,0,3,2] */, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E /* quad_perm [2,3,0,1] */, 0xF, 0xF, false);
    return v;
}

// Reserves HOLD_KB kilobytes of LDS in the kernel that calls it and never uses them: the only
// effect is that fewer blocks fit into a compute unit's LDS, i.e. a cap on the traffic a unit
// keeps in flight (see step_kernels.hpp for why that matters).  `never` must be false at run
// time; the dead store through `sink` only keeps the compiler from dropping the array.
template <int HOLD_KB>
__device__ __forceinline__ void reserve_lds(bool never, uint32_t *sink) {
    if constexpr (HOLD_KB > 0) {
        __shared__ uint32_t hold[HOLD_KB * 256];
        if (never) {
            hold[threadIdx.x] = threadIdx.x;
            sink[threadIdx.x] = hold[threadIdx.x ^ 1];
        }
    }
}

// Which tile a block takes.  Blocks go to the eight compute dies (XCDs) in turn, so block b and b + 8 share one.  With
// CHUNK > 0 a die takes 2^CHUNK neighbouring tiles before the next one's turn; what does not fill eight
// such runs is taken in order.
template <uint32_t CHUNK>
__device__ __forceinline__ uint32_t die_tile(uint32_t block, uint32_t n_tiles) {
    if constexpr (CHUNK == 0) return block;
    const uint32_t turn = block >> 3;
    const uint32_t tile = ((turn >> CHUNK << 3 | (block & 7u)) << CHUNK) | (turn & ((1u << CHUNK) - 1u));
    return block < (n_tiles >> (CHUNK + 3) << (CHUNK + 3)) ? tile : block;
}

// kernel argument block: M device pointers by value (no table in memory)
template <int N>
struct PtrTable {
    const void *g[N];
    float *m[N];           // all NULL when there is no momentum
    uint32_t *packed[N];   // all NULL when per-worker bits are not wanted
};

}  // namespace ss
