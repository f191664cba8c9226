// Device-side pieces shared by the kernels of libqesgd (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qesgd_internal.h"

namespace qesgd {

// Three-way xor in one v_bitop3 (truth table of a ^ b ^ c).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).  counter = (c0, c1, c2, c3), key = (k0, k1).
// One round: two 32x32->64 products; the high halves are mixed with the other two counter words
// and the key, the key advances by the Weyl constants.  The key is wave-uniform in every kernel
// here, so its schedule lives in scalar registers; the 64-bit products are single v_mad_u64_u32.
// Where c1 and c2 are uniform as well (a tile's group numbers share the high word), the first round's
// second product, its mix and the second round's first product are scalar too: 18 of the 20 vector
// products and 18 of the 20 mixes remain (the mix of round one is written with plain xors for that).
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&o)[4]) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t pa = (uint64_t)0xD2511F53u * c0;
        const uint64_t pb = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = r == 0 ? (uint32_t)(pb >> 32) ^ c1 ^ k0 : xor3((uint32_t)(pb >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(pa >> 32), c3, k1);
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    o[0] = c0; o[1] = c1; o[2] = c2; o[3] = c3;
}

// The 16-bit variate of the e-th of the 8 coordinates served by one call: word e/2, low half
// for even e, high half for odd e.
__device__ __forceinline__ uint32_t variate16(const uint32_t (&o)[4], int e) {
    const uint32_t word = o[e >> 1];
    return (e & 1) ? (word >> 16) : (word & 0xFFFFu);
}

// ---------------------------------------------------------------------------
// Streams of fp32 vectors.  Every vector of a round is touched once, so its 128-bit accesses carry
// the non-temporal policy: a line is the first to leave the caches and does not push out what will
// be read again.  Measured on 4.4 GB: reading 7.1 against 6.5 TB/s, reading plus the two packed
// planes of one level bit 6.6 against 5.7 TB/s, copying 6.6 against 6.25 TB/s.  The policy pays
// only when one instruction takes whole lines: with a lane owning 32 consecutive bytes (two loads
// that share every line) it costs instead, 5.1 against 5.7 TB/s.
//
// So a 512-coordinate chunk moves as two instructions of a contiguous KiB each, and the lane that
// needs coordinates 8l..8l+7 gets them by exchange: in each half of the chunk lane l < 32 moves
// float4 number 2l and lane 32 + l float4 number 2l + 1, and v_permlane32_swap (which swaps the
// upper lanes of its first operand with the lower lanes of its second) turns the two halves into
// 8 consecutive coordinates per lane, or back: 4 instructions and no LDS.
// ---------------------------------------------------------------------------
typedef float vec4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ vec4 load_stream(const float* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const vec4*>(p));
}
__device__ __forceinline__ void store_stream(float* p, const vec4& v) {
    __builtin_nontemporal_store(v, reinterpret_cast<vec4*>(p));
}
__device__ __forceinline__ vec4 load_cached(const float* p) { return *reinterpret_cast<const vec4*>(p); }
template <bool CACHED>
__device__ __forceinline__ vec4 load_as(const float* p) { return CACHED ? load_cached(p) : load_stream(p); }
template <bool CACHED>
__device__ __forceinline__ void store_as(float* p, const vec4& v) {
    if (CACHED) *reinterpret_cast<vec4*>(p) = v;
    else store_stream(p, v);
}

// CH x 512 coordinates of a vector, one float4 of each half chunk per lane, with either policy.
template <int CH, bool CACHED>
__device__ __forceinline__ void load_halves_as(const float* __restrict__ p, vec4 (&a)[CH], vec4 (&b)[CH]) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        a[c] = CACHED ? load_cached(p + c * kChunk) : load_stream(p + c * kChunk);
        b[c] = CACHED ? load_cached(p + c * kChunk + kChunk / 2) : load_stream(p + c * kChunk + kChunk / 2);
    }
}
// The policy chosen at run time; the condition is uniform.  The empty asm statements keep the compiler from
// merging the two arms into one set of loads, which would drop the policy.  Not for loads that are to stay in
// flight over other work: behind the arms the compiler no longer knows how many loads are younger than the
// ones it needs, and waits for all of them.
template <int CH>
__device__ __forceinline__ void load_halves(const float* __restrict__ p, bool cached, vec4 (&a)[CH], vec4 (&b)[CH]) {
    if (cached) {
        asm volatile("; cached");
        load_halves_as<CH, true>(p, a, b);
        asm volatile("; cached end");
    } else {
        load_halves_as<CH, false>(p, a, b);
    }
}

// Offset of this lane's float4 inside a half chunk (256 coordinates).
__device__ __forceinline__ uint32_t half_offset(uint32_t lane) { return (lane & 31u) * 8u + (lane >> 5) * 4u; }

// One float4 of each half per lane <-> 8 consecutive coordinates per lane.
__device__ __forceinline__ void halves_to_lane(const vec4& a, const vec4& b, float (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[i]), __float_as_uint(b[i]), false, false);
        v[i] = __uint_as_float(r[0]);
        v[4 + i] = __uint_as_float(r[1]);
    }
}
__device__ __forceinline__ void lane_to_halves(const float (&v)[8], vec4& a, vec4& b) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[4 + i]), false, false);
        a[i] = __uint_as_float(r[0]);
        b[i] = __uint_as_float(r[1]);
    }
}

// The first `count` of those coordinates: a float4 that is not wholly inside is taken element by element
// (stores leave the rest of it alone, loads give 0 there).
template <bool CACHED>
__device__ __forceinline__ vec4 load_part(const float* __restrict__ p, uint32_t at, uint32_t count) {
    vec4 r = {0.0f, 0.0f, 0.0f, 0.0f};
    if (at + 4u <= count) {
        r = CACHED ? load_cached(p + at) : load_stream(p + at);
    } else {
#pragma unroll
        for (uint32_t e = 0; e < 3; ++e)
            if (at + e < count) r[e] = p[at + e];
    }
    return r;
}
__device__ __forceinline__ void store_part(float* __restrict__ p, uint32_t at, uint32_t count, const vec4& v) {
    if (at + 4u <= count) {
        *reinterpret_cast<vec4*>(p + at) = v;
    } else {
#pragma unroll
        for (uint32_t e = 0; e < 3; ++e)
            if (at + e < count) p[at + e] = v[e];
    }
}
// CH x 512 coordinates of a vector from p on, one float4 of each half chunk per lane; at the ragged end of the
// vector (FULL = false) the first `count`, the rest 0, with the ordinary policy.
template <int CH, bool CACHED = true>
__device__ __forceinline__ void load_ragged(const float* __restrict__ p, uint32_t lane, uint32_t count, vec4 (&a)[CH], vec4 (&b)[CH]) {
    const uint32_t h = half_offset(lane);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        a[c] = load_part<CACHED>(p, h + c * kChunk, count);
        b[c] = load_part<CACHED>(p, h + c * kChunk + kChunk / 2, count);
    }
}
template <int CH, bool FULL>
__device__ __forceinline__ void load_chunks(const float* __restrict__ p, uint32_t lane, uint32_t count, bool cached,
                                            vec4 (&a)[CH], vec4 (&b)[CH]) {
    if (FULL) load_halves<CH>(p + half_offset(lane), cached, a, b);
    else load_ragged<CH>(p, lane, count, a, b);
}
template <int CH, bool FULL, bool CACHED>
__device__ __forceinline__ void load_chunks_as(const float* __restrict__ p, uint32_t lane, uint32_t count, vec4 (&a)[CH], vec4 (&b)[CH]) {
    if (FULL) load_halves_as<CH, CACHED>(p + half_offset(lane), a, b);
    else load_ragged<CH>(p, lane, count, a, b);
}
// One float4 of each half of 512 coordinates, back.
template <bool FULL>
__device__ __forceinline__ void store_chunk(float* __restrict__ p, uint32_t lane, uint32_t count, const vec4& a, const vec4& b) {
    const uint32_t h = half_offset(lane);
    if (FULL) {
        store_stream(p + h, a);
        store_stream(p + h + kChunk / 2, b);
    } else {
        store_part(p, h, count, a);
        store_part(p, h + kChunk / 2, count, b);
    }
}

// Tile of workgroup b.  Workgroups are handed to the 8 XCDs round-robin by id, so consecutive ids
// would spread every stretch of memory over all of them.  Groups of 2^lg tiles (256 KB of input, set
// by the host) go to one XCD instead: its reads and packed writes are then one run of addresses each
// (M = 1, bucket 4096: 0.70 against 0.77 ms at 1.07 G coordinates; groups of 64 K .. 1 M coordinates
// are within 2% of each other).  What is left over at the end stays in order.
// Workgroup 0 takes the last tile, the ragged one where there is one: its guarded code is the longest
// way through the kernel and would otherwise run on alone at the end.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t tiles, uint32_t lg) {
    --tiles;
    if (b == 0) return tiles;
    --b;
    if (b >= ((tiles >> (lg + 3u)) << (lg + 3u))) return b;
    const uint32_t r = b >> 3;
    return ((((r >> lg) << 3) | (b & 7u)) << lg) | (r & ((1u << lg) - 1u));
}
inline uint32_t xcd_group_log2(uint64_t tile) {
    uint32_t lg = 0;
    while ((tile << lg) < 65536u) ++lg;
    return lg;
}

}  // namespace qesgd
