// Device code of the quantiser shared by the translation units that launch it (not installed):
// the kernel parameter block, the cross-lane tree, rounding and packing of a lane's 8 coordinates,
// a wave on any bucket and the straight-line tile of the power-of-two-bucket kernels.
#pragma once

#include <type_traits>

#include "qesgd_aggregate_device.h"
#include "qesgd_device.h"
#include "qesgd_internal.h"

namespace qesgd {

// In the order that a kernel reads it in: a field in the middle that moved the rest cost calls of one or two short kernels
// 0.6 us (d = 0.9 M, K = 4, s = 16, bucket 65536 7.2 -> 7.8 us).  New ones go to the end.
struct QParams {
    const float* x;
    const float* center;
    unsigned char* packed;
    float* workspace;
    uint64_t x_stride;
    uint64_t packed_stride;
    uint64_t d;
    uint64_t B;
    uint64_t nb;
    uint64_t norms_off, signs_off, levels_off;
    uint32_t log2N;
    uint32_t log2_waves;         // general kernels: waves per workgroup
    uint32_t full_tiles;         // fast kernels: tiles per worker that lie wholly inside the vector; general ones: all
    uint32_t tail_tiles;         // fast quantize kernel: ragged tiles per worker after those (0 or 1)
    uint32_t group_workers;      // workers covered by this launch
    uint32_t xcd_group;          // fast quantize kernels: log2 of the tiles that one XCD takes in a row
    uint32_t ws_tiles_per_worker;  // partial sums: workspace entries per worker (nb * N / 4096)
    bool merged;                 // last pass: finish the tree from the partial sums (see wave_total)
    uint64_t data_tiles;         // partial sums: 4096-slot tiles of a worker that hold coordinates
    uint32_t key0, key1;
    uint32_t round;
    uint32_t worker0;
    float smax;
    bool x_cached;               // read the vectors with the ordinary cache policy
    bool codes_cached;           // write the level planes with the ordinary cache policy
    bool ragged_cached;          // x_cached where a wave of the general kernels is ragged
    bool six_waves;              // host only: see stream_lds
};

// Kernel parameters of a quantise call, and the first launches of the dense two-pass path (qesgd_quantize.hip).
QParams quantize_params(const Shape& sh, const QuantizeArgs& a);
int launch_dense_norms(QParams& p, const Shape& sh, const QuantizeArgs& a);

namespace {


// ---------------------------------------------------------------------------
// Cross-lane helpers.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
    return __uint_as_float(dpp_u32<CTRL>(__float_as_uint(x)));
}
constexpr int kDppXor1 = 0xB1;          // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;          // quad_perm [2,3,0,1]
constexpr int kDppQuadLane0 = 0x00;     // quad_perm [0,0,0,0]: lane 0 of the quad to all four
constexpr int kDppHalfMirror = 0x141;   // lane l -> 7 - l inside each 8: the other quad
constexpr int kDppRowMirror = 0x140;    // lane l -> 15 - l inside each 16: the other 8

template <int KIND>
__device__ __forceinline__ float combine(float a, float b) {
    if (KIND == QESGD_NORM_L2) return a + b;
    return fmaxf(a, b);
}

// The two halves of an exchange between 16-lane rows (lanes l and l ^ 16) or
// between wave halves (l and l ^ 32): v_permlane16_swap / v_permlane32_swap hand
// every lane its own row's value and the partner row's value, in some order;
// the combine is commutative, so the order does not matter.
template <int KIND>
__device__ __forceinline__ float combine_xor16(float t) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return combine<KIND>(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int KIND>
__device__ __forceinline__ float combine_xor32(float t) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return combine<KIND>(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Butterfly over the lanes that share a bucket (lanes_per_bucket = 1..64, a power
// of two, wave-uniform).  The mirror steps fetch "the other half" because after
// the previous steps all lanes of a half hold the same value; a + b == b + a, so
// every lane ends with the tree sum.
template <int KIND>
__device__ __forceinline__ float lane_butterfly(float t, uint32_t lanes_per_bucket) {
    if (lanes_per_bucket > 1) t = combine<KIND>(t, dpp_f32<kDppXor1>(t));
    if (lanes_per_bucket > 2) t = combine<KIND>(t, dpp_f32<kDppXor2>(t));
    if (lanes_per_bucket > 4) t = combine<KIND>(t, dpp_f32<kDppHalfMirror>(t));
    if (lanes_per_bucket > 8) t = combine<KIND>(t, dpp_f32<kDppRowMirror>(t));
    if (lanes_per_bucket > 16) t = combine_xor16<KIND>(t);
    if (lanes_per_bucket > 32) t = combine_xor32<KIND>(t);
    return t;
}

template <int KIND>
__device__ __forceinline__ float lane_tree(const float (&v)[8]) {
    if (KIND == QESGD_NORM_L2) {
        const float q0 = v[0] * v[0], q1 = v[1] * v[1], q2 = v[2] * v[2], q3 = v[3] * v[3];
        const float q4 = v[4] * v[4], q5 = v[5] * v[5], q6 = v[6] * v[6], q7 = v[7] * v[7];
        return ((q0 + q1) + (q2 + q3)) + ((q4 + q5) + (q6 + q7));
    }
    return fmaxf(fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))),
                 fmaxf(fmaxf(fabsf(v[4]), fabsf(v[5])), fmaxf(fabsf(v[6]), fabsf(v[7]))));
}

// The same in-lane tree over 8 values that are already partial results (no squaring).
template <int KIND>
__device__ __forceinline__ float lane_tree_of_partials(const float (&q)[8]) {
    return combine<KIND>(combine<KIND>(combine<KIND>(q[0], q[1]), combine<KIND>(q[2], q[3])),
                         combine<KIND>(combine<KIND>(q[4], q[5]), combine<KIND>(q[6], q[7])));
}

// Pairwise tree over up to 16 wave totals parked in LDS; entries beyond `count`
// are +0 (adding +0 is exact, so the padded tree equals the tree over `count`).
// `sm` must have 32 readable floats: a hoisted read of sm[base + r] stays inside.
template <int KIND>
__device__ __forceinline__ float lds_tree16(const float* sm, uint32_t base, uint32_t count) {
    float a[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] = ((uint32_t)r < count) ? sm[base + r] : 0.0f;
#pragma unroll
    for (int w = 1; w < 16; w <<= 1) {
#pragma unroll
        for (int r = 0; r < 16; r += 2 * w) a[r] = combine<KIND>(a[r], a[r + w]);
    }
    return a[0];
}

// The rest of a bucket's tree by one wave, for at most 1024 partial sums of which the first `valid` were
// written (the others are +0, the identity of both combines): a lane takes 16 consecutive ones, index
// bits 0-3, the lanes bits 4-9.  P, a power of two >= 16, entries are readable.
constexpr uint32_t kMergedLeaves = 1024;
template <int KIND>
__device__ __forceinline__ float wave_total(const float* __restrict__ ws, uint32_t P, uint32_t valid, uint32_t lane) {
    const uint32_t first = lane * 16u;
    const float* __restrict__ src = ws + (first < P ? first : 0u);
    float q[16];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const vec4 a = load_cached(src + 4 * i);
#pragma unroll
        for (int e = 0; e < 4; ++e) q[4 * i + e] = first + (uint32_t)(4 * i + e) < valid ? a[e] : 0.0f;
    }
#pragma unroll
    for (int w = 1; w < 16; w <<= 1) {
#pragma unroll
        for (int r = 0; r < 16; r += 2 * w) q[r] = combine<KIND>(q[r], q[r + w]);
    }
    return lane_butterfly<KIND>(q[0], 64);
}

// ---------------------------------------------------------------------------
// Bucket scale.
// ---------------------------------------------------------------------------
// Correctly rounded square root and quotient for operands far from the ends of the exponent range:
// the hardware estimate and the correction steps of the general expansions without their operand
// scaling and special cases, which the ranges of their callers leave out (norms of 2^-60 to 2^60, totals
// of 2^-90 to 2^120); the tests compare codes and scales with IEEE arithmetic at both ends of these ranges.
__device__ __forceinline__ float sqrt_in_range(float x) {
    const float s = __builtin_amdgcn_sqrtf(x);
    const float down = __uint_as_float(__float_as_uint(s) - 1u), up = __uint_as_float(__float_as_uint(s) + 1u);
    const float rd = __builtin_fmaf(-down, s, x), ru = __builtin_fmaf(-up, s, x);
    const float r = rd <= 0.0f ? down : s;
    return ru > 0.0f ? up : r;
}
__device__ __forceinline__ float quotient_in_range(float a, float b) {
    float r = __builtin_amdgcn_rcpf(b);
    r = __builtin_fmaf(__builtin_fmaf(-b, r, 1.0f), r, r);
    float q = a * r;
    q = __builtin_fmaf(__builtin_fmaf(-b, q, a), r, q);
    return __builtin_fmaf(__builtin_fmaf(-b, q, a), r, q);
}
__device__ __forceinline__ float inverse_step(float norm, float smax) {
    float inv = smax / norm;
    if (!(inv < INFINITY)) inv = 0.0f;     // norm 0 (or reciprocal overflow): every level is 0
    return inv;
}

// How the buckets of a wave are scaled.  direct (the same for the whole wave): every norm is in
// [2^-60, 2^60] and mul = fl(smax/norm) * 2^(32-M), the form that ordinary buckets take (see
// round_and_pack); otherwise mul is not used.
struct Scale {
    float norm, mul;
    bool direct;
};

__device__ __forceinline__ bool wave_all(bool x) { return __builtin_amdgcn_ballot_w64(!x) == 0; }

// No NaN among a lane's coordinates.  The L2 norm of a bucket with a NaN is a NaN itself, but a maximum
// passes over it, so under the max norm the direct form has to look (4 compares per 8 coordinates).
template <int KIND>
__device__ __forceinline__ bool no_nan(const float (&v)[8]) {
    if (KIND == QESGD_NORM_L2) return true;
    return !(__builtin_isunordered(v[0], v[1]) || __builtin_isunordered(v[2], v[3]) ||
             __builtin_isunordered(v[4], v[5]) || __builtin_isunordered(v[6], v[7]));
}

template <int M>
__device__ __forceinline__ Scale scale_of_norm(float norm) {
    constexpr float smax = (float)((1u << M) - 1u);
    Scale sc;
    sc.norm = norm;
    sc.direct = wave_all(norm >= 0x1p-60f && norm <= 0x1p60f);
    sc.mul = quotient_in_range(smax * (float)(1ull << (32 - M)), norm);
    return sc;
}

// The scale of a bucket whose tree total (L2) or maximum is t.
template <int M, int KIND>
__device__ __forceinline__ Scale scale_of_total(float t) {
    if (KIND != QESGD_NORM_L2) return scale_of_norm<M>(t);
    constexpr float smax = (float)((1u << M) - 1u);
    Scale sc;
    sc.direct = wave_all(t >= 0x1p-90f && t <= 0x1p120f);
    sc.norm = sc.direct ? sqrt_in_range(t) : sqrtf(t);
    sc.mul = quotient_in_range(smax * (float)(1ull << (32 - M)), sc.norm);
    return sc;
}

// ---------------------------------------------------------------------------
// Rounding and in-lane packing of the 8 coordinates of a lane.
//   fixed = trunc(min(|v| * inv, smax) * 2^16) = floor(a) * 2^16 + trunc(frac(a) * 2^16)
//   level = (fixed + r16) >> 16        (the carry out of the low half rounds up)
// bits[] receives the 8*M level bits (M = 1: low byte, M = 2: low half, M = 4: one word, M = 8: two
// words, M = 16: four words; M = 3, 5, 6, 7: the low 8*M bits of bits[0..1] read as one 64-bit string).
//
// Direct form, 5 instructions per coordinate with the sign and the packing (10 before, which showed as
// 0.62 ms of vector issue on d = 138 M, K = 8, s = 2):
//   p = fma(v, mul, +0)       the product with its sign; the +0 turns -0 * mul into +0, so the sign bit
//                             of p is [v < 0] also for v = -0, and changes no other product
//   y = trunc(|p|) + r16 * 2^(16-M), saturating (v_mad_u32_u16 picks either half of the random word)
//   level = the top M bits of y, sign = the top bit of p; one v_alignbit appends each to its string.
// The scale carries 2^(32-M) instead of 2^16, so that the level lands in the top bits: the 16-M bits of
// trunc(|p|) below the random number's lowest bit cannot carry.  Scaling by a power of two commutes
// with rounding, and a product that underflows truncates to 0 either way.
// The minimum with smax is not needed: norm >= |v| (the tree total is at least fl(v^2), and sqrt is
// monotonic with sqrt(fl(v^2)) = |v|, away from underflow), so |p| exceeds smax * 2^(32-M) by at most
// the last place of the product; for M <= 7 that is less than 2^(16-M) and never carries, and for
// M = 8, 16 the saturating sum keeps the top level.
// A bucket whose norm is outside [2^-60, 2^60] (zero buckets among them) or a wave that holds a NaN takes
// the formula as it stands.
// ---------------------------------------------------------------------------
template <int HALF>
__device__ __forceinline__ uint32_t add_variate(uint32_t word, uint32_t weight, uint32_t a) {
    uint32_t y;
    if (HALF == 0) asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[0,0,0,0] clamp" : "=v"(y) : "v"(word), "s"(weight), "v"(a));
    else asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0] clamp" : "=v"(y) : "v"(word), "s"(weight), "v"(a));
    return y;
}

// Level fields of four coordinates, level in the top M bits of each y (M < 8: 4*M bits; M = 8: a word).
template <int M>
__device__ __forceinline__ uint32_t pack4(const uint32_t* y) {
    if (M == 8) {
        const uint32_t lo = __builtin_amdgcn_perm(y[1], y[0], 0x0C0C0703u);     // byte 3 of each
        const uint32_t hi = __builtin_amdgcn_perm(y[3], y[2], 0x07030C0Cu);
        return lo | hi;
    }
    uint32_t w = y[3] >> (32 - M);
#pragma unroll
    for (int e = 2; e >= 0; --e) w = __builtin_amdgcn_alignbit(w, y[e], 32 - M);
    return w;
}

template <int M>
__device__ __forceinline__ void round_and_pack(const float (&v)[8], const uint32_t (&rnd)[4], const Scale& sc,
                                               uint32_t& sign_byte, uint32_t (&bits)[4]) {
    uint32_t y[8], sb;                                   // level in the top M bits of y
    if (sc.direct) {
        const uint32_t weight = 1u << (16 - M);
        uint32_t p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float pe = __builtin_fmaf(v[e], sc.mul, 0.0f);
            p[e] = __float_as_uint(pe);
            const uint32_t a = (uint32_t)fabsf(pe);
            y[e] = (e & 1) ? add_variate<1>(rnd[e >> 1], weight, a) : add_variate<0>(rnd[e >> 1], weight, a);
        }
        sb = p[7] >> 31;
#pragma unroll
        for (int e = 6; e >= 0; --e) sb = __builtin_amdgcn_alignbit(sb, p[e], 31);
    } else {
        constexpr float smax = (float)((1u << M) - 1u);
        // the product with 2^16 is folded into the scale where it is finite
        const float inv = inverse_step(sc.norm, smax);
        const bool fold = inv * 65536.0f < INFINITY;
        const float mul = fold ? inv * 65536.0f : inv, cap = fold ? smax * 65536.0f : smax, post = fold ? 1.0f : 65536.0f;
        sb = 0;
#pragma unroll
        for (int e = 7; e >= 0; --e) {
            const float a = fminf(fabsf(v[e]) * mul, cap) * post;
            y[e] = (((uint32_t)a + variate16(rnd, e)) >> 16) << (32 - M);
            sb = sb + sb + (v[e] < 0.0f ? 1u : 0u);
        }
    }
    sign_byte = sb;
    bits[0] = bits[1] = bits[2] = bits[3] = 0;
    if constexpr (M == 8) {
        bits[0] = pack4<M>(y);
        bits[1] = pack4<M>(y + 4);
    } else if constexpr (M == 16) {
#pragma unroll
        for (int q = 0; q < 4; ++q) bits[q] = __builtin_amdgcn_perm(y[2 * q + 1], y[2 * q], 0x07060302u);
    } else if constexpr (M <= 4 && M != 3) {
        uint32_t w = y[7] >> (32 - M);
#pragma unroll
        for (int e = 6; e >= 0; --e) w = __builtin_amdgcn_alignbit(w, y[e], 32 - M);
        bits[0] = w;
    } else {                                              // 8*M = 24..56 bits: one 64-bit string
        const uint64_t w = (uint64_t)pack4<M>(y) | ((uint64_t)pack4<M>(y + 4) << (4 * M));
        bits[0] = (uint32_t)w;
        bits[1] = (uint32_t)(w >> 32);
    }
}

// Cross-lane assembly of words and the stores, for a lane whose 8 coordinates
// start at coordinate i (a multiple of 8) of which nvalid (0..8) exist.
// sign_words / level_words point at word 0 of the planes.
template <int M>
__device__ __forceinline__ void store_codes(uint32_t* __restrict__ sign_words, uint32_t* __restrict__ level_words,
                                            uint64_t i, uint32_t nvalid, uint32_t lane,
                                            uint32_t sign_byte, const uint32_t (&bits)[4]) {
    {
        uint32_t w = sign_byte << (8u * (lane & 3u));
        w |= dpp_u32<kDppXor1>(w);
        w |= dpp_u32<kDppXor2>(w);
        if ((lane & 3u) == 0u && nvalid > 0) sign_words[i >> 5] = w;
    }
    if (M == 1) {
        uint32_t w = bits[0] << (8u * (lane & 3u));
        w |= dpp_u32<kDppXor1>(w);
        w |= dpp_u32<kDppXor2>(w);
        if ((lane & 3u) == 0u && nvalid > 0) level_words[i >> 5] = w;
    } else if (M == 2) {
        uint32_t w = bits[0] << (16u * (lane & 1u));
        w |= dpp_u32<kDppXor1>(w);
        if ((lane & 1u) == 0u && nvalid > 0) level_words[i >> 4] = w;
    } else if (M == 4) {
        if (nvalid > 0) level_words[i >> 3] = bits[0];
    } else if (M == 3 || M == 5 || M == 6 || M == 7) {
        // The 32 coordinates of a quad fill M whole words; lane j's 8*M bits start at bit
        // 8*M*j of that block.  Every lane shifts its string into each of the M words, the
        // quad ORs them, and lane j stores words j and j+4 of the block (those that hold a
        // coordinate of the vector).
        const uint32_t j = lane & 3u;
        uint32_t nq = nvalid;
        nq += dpp_u32<kDppXor1>(nq);
        nq += dpp_u32<kDppXor2>(nq);
        const uint32_t nwords = (nq * (uint32_t)M + 31u) >> 5;
        const uint64_t i_quad = (uint64_t)dpp_u32<kDppQuadLane0>((uint32_t)i) |
                                ((uint64_t)dpp_u32<kDppQuadLane0>((uint32_t)(i >> 32)) << 32);
        const uint64_t v = (uint64_t)bits[0] | ((uint64_t)bits[1] << 32);
        const int at = 8 * M * (int)j;
        uint32_t first = 0, second = 0;
#pragma unroll
        for (int q = 0; q < M; ++q) {
            const int sh = at - 32 * q;                   // where the string starts relative to word q
            uint32_t c = 0;
            if (sh >= 0 && sh < 32) c = (uint32_t)v << sh;
            else if (sh < 0 && sh > -64) c = (uint32_t)(v >> (-sh));
            c |= dpp_u32<kDppXor1>(c);
            c |= dpp_u32<kDppXor2>(c);
            if (q < 4) { if (j == (uint32_t)q) first = c; }
            else { if (j == (uint32_t)(q - 4)) second = c; }
        }
        uint32_t* __restrict__ dst = level_words + (i_quad >> 5) * (uint64_t)M;
        if (j < nwords) dst[j] = first;
        if (M > 4 && j + 4u < nwords) dst[j + 4u] = second;
    } else if (M == 8) {
        if (nvalid == 8) {
            *reinterpret_cast<uint2*>(level_words + (i >> 2)) = make_uint2(bits[0], bits[1]);
        } else {
            if (nvalid > 0) level_words[i >> 2] = bits[0];
            if (nvalid > 4) level_words[(i >> 2) + 1] = bits[1];
        }
    } else {
        if (nvalid == 8) {
            *reinterpret_cast<uint4*>(level_words + (i >> 1)) = make_uint4(bits[0], bits[1], bits[2], bits[3]);
        } else {
            if (nvalid > 0) level_words[i >> 1] = bits[0];
            if (nvalid > 2) level_words[(i >> 1) + 1] = bits[1];
            if (nvalid > 4) level_words[(i >> 1) + 2] = bits[2];
            if (nvalid > 6) level_words[(i >> 1) + 3] = bits[3];
        }
    }
}

// The codes of a lane's 8 coordinates where all of them exist: lane group `idx` of the planes that
// start at the (uniform) bytes signs and levels.  A lane's sign bits are one byte and its level bits M,
// so widths that divide 32 need no exchange between lanes: 64 lanes write consecutive bytes.  A wave's
// level bits fill whole lines from M = 2 on and leave with the non-temporal policy (M = 8, buckets of
// 512: 0.81 against 0.94 ms at 1.07 G coordinates); the 64-byte halves of a line that one-bit planes
// are written in meet in the L2 and keep the ordinary policy (0.72 against 0.75 ms).
template <int M, bool CACHED>
__device__ __forceinline__ void store_codes_full(unsigned char* __restrict__ signs, unsigned char* __restrict__ levels,
                                                 uint32_t idx, uint32_t sign_byte, const uint32_t (&bits)[4]) {
    typedef uint32_t uvec2 __attribute__((ext_vector_type(2)));
    typedef uint32_t uvec4 __attribute__((ext_vector_type(4)));
    signs[idx] = (unsigned char)sign_byte;
    if constexpr (M == 1) {
        levels[idx] = (unsigned char)bits[0];
    } else {
        typedef std::conditional_t<M == 2, unsigned short, std::conditional_t<M == 4, uint32_t, std::conditional_t<M == 8, uvec2, uvec4>>> field;
        field f;
        if constexpr (M == 8) f = uvec2{bits[0], bits[1]};
        else if constexpr (M == 16) f = uvec4{bits[0], bits[1], bits[2], bits[3]};
        else f = (field)bits[0];
        field* dst = reinterpret_cast<field*>(levels + idx * (uint32_t)M);
        if (CACHED) *dst = f;
        else __builtin_nontemporal_store(f, dst);
    }
}

// The same for the CH chunks of a wave that follow each other from lane group idx0 on.  One branch behind
// all chunks: a branch per chunk would keep the chunks' arithmetic apart (528 against 504 us for the two
// calls of a round at d = 25.6 M, K = 16, s = 256, bucket 8192).
template <int M, int CH>
__device__ __forceinline__ void store_chunks(unsigned char* __restrict__ signs, unsigned char* __restrict__ levels, uint32_t idx0,
                                             bool cached, const uint32_t (&sign_byte)[CH], const uint32_t (&bits)[CH][4]) {
    if (M > 1 && cached) {
        asm volatile("; cached");                         // keeps the arms apart (see load_halves)
#pragma unroll
        for (int c = 0; c < CH; ++c) store_codes_full<M, true>(signs, levels, idx0 + (uint32_t)c * kWaveSize, sign_byte[c], bits[c]);
        asm volatile("; cached end");
    } else {
#pragma unroll
        for (int c = 0; c < CH; ++c) store_codes_full<M, false>(signs, levels, idx0 + (uint32_t)c * kWaveSize, sign_byte[c], bits[c]);
    }
}

// Level strings of 512 consecutive coordinates for the widths that do not divide 32: the lanes' M bytes each meet in
// LDS private to the wave and leave as consecutive 16-byte pieces.  words: the first of 16 * M, on any word.  mine: the
// wave's kStringBytes of LDS.  Chunk by chunk and with the ordinary policy (two chunks at a time: d = 3.5 M, K = 8, s = 128,
// bucket 8192 27.7 us, 26.3 one by one; byte by byte: as
// unaligned words d = 49 M, K = 8, s = 128, bucket 8192 336 us, 326 as bytes; non-temporal: d = 10 M, K = 8, s = 64, one bucket, gradient round 164 us, 157).
template <int M>
constexpr uint32_t kStringBytes = 32 % M == 0 ? 0 : kWaveSize * M;
template <int M>
__device__ __forceinline__ void store_levels_lds(unsigned char* mine, uint32_t* __restrict__ words, uint32_t lane, const uint32_t (&bits)[4]) {
    typedef uint32_t uvec4 __attribute__((ext_vector_type(4)));
    typedef uvec4 anywhere __attribute__((aligned(4)));
#pragma unroll
    for (int j = 0; j < M; ++j) mine[lane * (uint32_t)M + j] = (unsigned char)(bits[j >> 2] >> (8 * (j & 3)));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane < 4u * M) reinterpret_cast<anywhere*>(words)[lane] = *reinterpret_cast<const uvec4*>(mine + lane * 16u);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();                      // the next chunk overwrites the area
}

// The codes of a wave's 512 consecutive coordinates from coordinate i0 (a multiple of 32) on.
template <int M>
__device__ __forceinline__ void store_whole(unsigned char* string, unsigned char* __restrict__ signs, unsigned char* __restrict__ levels, uint64_t i0,
                                            uint32_t lane, bool cached, uint32_t sign_byte, const uint32_t (&bits)[4]) {
    const uint64_t g0 = i0 / kLaneElems;
    if constexpr (32 % M == 0) {
        const uint32_t sb[1] = {sign_byte}, bt[1][4] = {{bits[0], bits[1], bits[2], bits[3]}};
        store_chunks<M, 1>(signs + g0, levels + g0 * M, lane, cached, sb, bt);
    } else {
        (signs + g0)[lane] = (unsigned char)sign_byte;
        store_levels_lds<M>(string, reinterpret_cast<uint32_t*>(levels + g0 * M), lane, bits);
    }
}

// Of the tile's `count` coordinates those from the wave's first on.
__device__ __forceinline__ uint32_t count_from(uint32_t count, uint32_t first) { return count > first ? count - first : 0u; }

// A wave's CH chunks of a tile into registers: xw / cw point at the wave's first coordinate.  All
// loads are issued before the first use.  `center` is read by every worker's workgroup of the tile,
// so it keeps the ordinary cache policy.
template <int CH, bool CENTER, bool FULL = true>
__device__ __forceinline__ void load_tile(const float* __restrict__ xw, const float* __restrict__ cw, uint32_t lane,
                                          bool x_cached, float (&v)[CH][8], uint32_t count = CH * kChunk) {
    vec4 a[CH], b[CH], ca[CH], cb[CH];
    load_chunks<CH, FULL>(xw, lane, count, x_cached, a, b);
    if (CENTER) load_chunks<CH, FULL>(cw, lane, count, true, ca, cb);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (CENTER) {
            a[c] -= ca[c];
            b[c] -= cb[c];
        }
        halves_to_lane(a[c], b[c], v[c]);
    }
}

// ---------------------------------------------------------------------------
// A wave on CH x 512 slots that hold consecutive coordinates, whatever the bucket's size.
// ---------------------------------------------------------------------------
// Where the wave's slots fall, worked out in scalar registers: `mine` coordinates (0: all padding) from coordinate
// i0 (a multiple of 32) on, in bucket `bucket`, in whose slots the wave is number `sub`.
struct WaveSpan {
    uint64_t bucket, i0;
    uint32_t sub, mine;
};

// max(0, min(left, most)).  In 32-bit comparisons: a uniform 64-bit one runs on the vector unit, and where its result
// served a branch and a selection the compiler lost the latter's condition (the selection took whatever carry was last).
__device__ __forceinline__ uint32_t clamp_left(int64_t left, uint32_t most) {
    const int32_t high = (int32_t)(left >> 32);
    const uint32_t low = (uint32_t)left;
    return high < 0 ? 0u : high > 0 || low > most ? most : low;
}

// unit: the wave's number in slot space.  Buckets are 2^lg waves.
template <int CH>
__device__ __forceinline__ WaveSpan wave_span(const QParams& p, uint64_t unit, uint32_t lg) {
    WaveSpan s;
    s.bucket = unit >> lg;
    s.sub = (uint32_t)unit & ((1u << lg) - 1u);
    const uint64_t j = (unit & ((1ull << lg) - 1u)) * (CH * kChunk), at = s.bucket * p.B + j;
    const uint32_t in_bucket = clamp_left((int64_t)(p.B - j), CH * kChunk), in_vector = clamp_left((int64_t)(p.d - at), CH * kChunk);
    s.mine = in_bucket < in_vector ? in_bucket : in_vector;
    s.i0 = s.mine ? at : 0;
    return s;
}
// The same where slots are coordinates (a bucket that is a power of two, or the only one); the bucket is left out.
template <int CH>
__device__ __forceinline__ WaveSpan wave_span_dense(const QParams& p, uint64_t unit) {
    WaveSpan s{};
    const uint64_t at = unit * (CH * kChunk);
    s.mine = clamp_left((int64_t)(p.d - at), CH * kChunk);
    s.i0 = s.mine ? at : 0;
    return s;
}

// The float4 of each half chunk that lie inside the first `whole` coordinates (a multiple of 4, not 0); h: half_offset.
template <int CH, bool CACHED>
__device__ __forceinline__ void load_inside(const float* __restrict__ p, uint32_t h, uint32_t whole, vec4 (&a)[CH], vec4 (&b)[CH]) {
#pragma unroll
    for (uint32_t c = 0; c < CH; ++c) {
        const uint32_t at = h + c * kChunk, ia = at < whole ? at : 0u, ib = at + kChunk / 2 < whole ? at + kChunk / 2 : 0u;
        a[c] = CACHED ? load_cached(p + ia) : load_stream(p + ia);
        b[c] = CACHED ? load_cached(p + ib) : load_stream(p + ib);
    }
}

// Worker k's coordinates of the span, 0 beyond it.
template <int CH, bool CENTER>
__device__ __forceinline__ void load_span(const QParams& p, uint32_t k, const WaveSpan& s, uint32_t lane, float (&v)[CH][8]) {
    const float* __restrict__ x = p.x + (uint64_t)k * p.x_stride + s.i0;
    const float* __restrict__ center = p.center + s.i0;
    if (s.mine == CH * kChunk) {
        load_tile<CH, CENTER>(x, center, lane, p.x_cached, v);
        return;
    }
    vec4 a[CH], b[CH], ca[CH], cb[CH];
    if constexpr (CENTER && CH == 2) {
        // A float4 that is not wholly inside is read at the wave's first coordinates and means nothing.  Behind a condition of
        // its lane (as below) a load waits for those before it, the center's for x's: d = 12 M, K = 1, s = 16, bucket 12000
        // 20.4 us, this 17.9.  (Without a center this is no faster, and with four chunks it takes 121 registers: d = 25.6 M, K = 4,
        // s = 256, bucket 20000, no center 123 / 143 us.)
        const uint32_t whole = s.mine & ~3u, h = half_offset(lane);
        if (whole != 0u) {
            if (p.ragged_cached) {
                asm volatile("; cached");                 // keeps the arms apart (see load_halves)
                load_inside<CH, true>(x, h, whole, a, b);
                asm volatile("; cached end");
            } else {
                load_inside<CH, false>(x, h, whole, a, b);
            }
            load_inside<CH, true>(center, h, whole, ca, cb);
        }
#pragma unroll
        for (uint32_t c = 0; c < CH; ++c) {
            const uint32_t at = h + c * kChunk;
            a[c] -= ca[c];
            b[c] -= cb[c];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[c][e] = at < whole ? a[c][e] : 0.0f;
                b[c][e] = at + kChunk / 2 < whole ? b[c][e] : 0.0f;
            }
            if (s.mine != whole) {                        // the vector ends off a float4 (buckets are multiples of 32)
#pragma unroll
                for (uint32_t e = 0; e < 3; ++e) {
                    const uint32_t i = whole + e;
                    if (at == whole && i < s.mine) a[c][e] = x[i] - center[i];
                    if (at + kChunk / 2 == whole && i < s.mine) b[c][e] = x[i] - center[i];
                }
            }
        }
    } else if (p.ragged_cached) {
        asm volatile("; cached");
        load_tile<CH, CENTER, false>(x, center, lane, true, v, s.mine);
        asm volatile("; cached end");
        return;
    } else {
        load_ragged<CH, false>(x, lane, s.mine, a, b);
        if (CENTER) load_ragged<CH, true>(center, lane, s.mine, ca, cb);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (CENTER) {
                a[c] -= ca[c];
                b[c] -= cb[c];
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) halves_to_lane(a[c], b[c], v[c]);
}

// The codes of CH x 512 coordinates that all exist, from coordinate i0 on, whose group numbers share their high word.
// string: kStringBytes<M> of LDS that are the wave's.
template <int M, int CH, int KIND>
__device__ __forceinline__ void encode_whole(const QParams& p, uint32_t k, uint64_t i0, uint32_t lane, unsigned char* string,
                                             const float (&v)[CH][8], const Scale (&sc)[CH]) {
    unsigned char* __restrict__ out = p.packed + (uint64_t)k * p.packed_stride;
    const uint64_t g0 = i0 / kLaneElems;
    uint32_t sign_byte[CH], bits[CH][4];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        uint32_t rnd[4];
        philox4x32_10((uint32_t)g0 + (uint32_t)c * kWaveSize + lane, (uint32_t)(g0 >> 32), p.worker0 + k, p.round, p.key0, p.key1, rnd);
        Scale own = sc[c];
        if (KIND != QESGD_NORM_L2) own.direct = own.direct && wave_all(no_nan<KIND>(v[c]));
        round_and_pack<M>(v[c], rnd, own, sign_byte[c], bits[c]);
        if constexpr (32 % M != 0)
            store_whole<M>(string, out + p.signs_off, out + p.levels_off, i0 + (uint32_t)c * kChunk, lane, p.codes_cached, sign_byte[c], bits[c]);
    }
    if constexpr (32 % M == 0) store_chunks<M, CH>(out + p.signs_off + g0, out + p.levels_off + g0 * M, lane, p.codes_cached, sign_byte, bits);
}

// The codes of a span.
template <int M, int CH, int KIND>
__device__ __forceinline__ void encode_span(const QParams& p, uint32_t k, const WaveSpan& s, uint32_t lane, unsigned char* string,
                                            const float (&v)[CH][8], const Scale (&sc)[CH]) {
    const uint64_t g0 = s.i0 / kLaneElems;
    if (s.mine == CH * kChunk && (uint32_t)g0 <= 0u - (uint32_t)CH * kWaveSize) {
        encode_whole<M, CH, KIND>(p, k, s.i0, lane, string, v, sc);
        return;
    }
    unsigned char* __restrict__ out = p.packed + (uint64_t)k * p.packed_stride;
    uint32_t sign_byte[CH], bits[CH][4];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (s.mine <= (uint32_t)c * kChunk) break;                               // no coordinate left
        const uint64_t g = g0 + (uint32_t)c * kWaveSize + lane;
        uint32_t rnd[4];
        philox4x32_10((uint32_t)g, (uint32_t)(g >> 32), p.worker0 + k, p.round, p.key0, p.key1, rnd);
        Scale own = sc[c];
        if (KIND != QESGD_NORM_L2) own.direct = own.direct && wave_all(no_nan<KIND>(v[c]));
        round_and_pack<M>(v[c], rnd, own, sign_byte[c], bits[c]);
        const uint32_t at = (uint32_t)c * kChunk + lane * kLaneElems, rest = count_from(s.mine, at);
        store_codes<M>(reinterpret_cast<uint32_t*>(out + p.signs_off), reinterpret_cast<uint32_t*>(out + p.levels_off), s.i0 + at,
                       rest < 8u ? rest : 8u, lane, sign_byte[c], bits[c]);
    }
}

// ---------------------------------------------------------------------------
// Lane by lane: buckets padded to 512 or less that are neither a power of two nor the only one, every wave of which
// holds padding.
// ---------------------------------------------------------------------------
// Where the 8 slots of a lane fall: bucket, first coordinate (a multiple of 8), 4 coordinates that exist, how many of
// the 8 are real coordinates (0..8), and whether they open the bucket.
struct LaneSpan {
    uint64_t bucket, i, safe;
    uint32_t nvalid;
    bool opens_bucket;
};

__device__ __forceinline__ LaneSpan lane_span(uint64_t slot, const QParams& p) {
    LaneSpan s{};
    const uint64_t N = 1ull << p.log2N;
    s.bucket = slot >> p.log2N;
    const uint64_t j = slot & (N - 1);
    uint64_t len = 0;
    if (s.bucket < p.nb) {
        const uint64_t rem = p.d - s.bucket * p.B;
        len = rem < p.B ? rem : p.B;
    }
    s.nvalid = j < len ? (uint32_t)((len - j) < 8 ? (len - j) : 8) : 0u;
    s.i = s.bucket * p.B + j;
    s.safe = len >= 4 ? s.i - j : 0;
    s.opens_bucket = (j == 0) && (s.bucket < p.nb);
    return s;
}

// The coordinates of a lane's slots, 0 beyond them: two float4, read from s.safe where they are not wholly inside, so that
// the loads of all chunks, and of the center behind them, are in flight together.  (A vector of several
// such buckets has more than 4.)
template <int CH, bool CENTER>
__device__ __forceinline__ void load_lanes(const QParams& p, uint32_t k, const LaneSpan (&span)[CH], float (&v)[CH][8]) {
    const float* __restrict__ x = p.x + (uint64_t)k * p.x_stride;
    vec4 a[CH], b[CH], ca[CH], cb[CH];
    bool end = false;                                     // the vector ends here, off a float4 (the same for the wave)
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const uint64_t ia = span[c].nvalid >= 4u ? span[c].i : span[c].safe, ib = span[c].nvalid == 8u ? span[c].i + 4u : span[c].safe;
        a[c] = load_cached(x + ia);
        b[c] = load_cached(x + ib);
        if (CENTER) {
            ca[c] = load_cached(p.center + ia);
            cb[c] = load_cached(p.center + ib);
        }
        end = end || !wave_all(span[c].nvalid == 0u || span[c].nvalid == 8u);
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (CENTER) {
            a[c] -= ca[c];
            b[c] -= cb[c];
        }
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) {
            v[c][e] = span[c].nvalid >= 4u ? a[c][e] : 0.0f;
            v[c][4 + e] = span[c].nvalid == 8u ? b[c][e] : 0.0f;
        }
        if (end) {
#pragma unroll
            for (uint32_t e = 0; e < 8; ++e) {
                const bool last = span[c].nvalid < 8u && e < span[c].nvalid && e >= (span[c].nvalid & 4u);
                if (last) v[c][e] = CENTER ? x[span[c].i + e] - p.center[span[c].i + e] : x[span[c].i + e];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Fast kernel.  Geometry per bucket size: tile = NW waves x CH chunks x 512.
// ---------------------------------------------------------------------------
template <int M, int LOG2N, bool CENTER = false>
struct Geo {
    // Chunks per wave and waves per workgroup, measured at 480 M coordinates with the non-temporal streams.  Two
    // chunks per wave, the more bytes in flight the better (one / two: M = 2, bucket 2048 361 / 341 us; M = 4,
    // 512 377 / 358; M = 8, 128 421 / 393; M = 8, 4096 408 / 394; four are slower, M = 1, bucket 4096 at 1.1 G
    // 860 / 811).  With a center its coordinates are held as well, and from M = 4 on neither is always better
    // (quantiser, one / two: 30 M, K = 8, M = 8, bucket 2048 248 / 259 us; 57 M, K = 2, M = 4, 4096 127 / 130; 58 M,
    // K = 4, M = 4, 4096 228 / 236; but 57 M, K = 8, M = 8, 512 490 / 450; 120 M, K = 4, M = 4, 4096 496 / 481; 16 M,
    // K = 16, M = 4, 4096 255 / 251): one.  The workgroup is as small as the bucket allows, but not one wave
    // (M = 4: the same; M = 1: slower).
    static constexpr int CH = LOG2N == 15 ? 4 : (CENTER && M > 2 && LOG2N < 13 ? 1 : 2);
    static constexpr int NW = (1 << LOG2N) / (CH * 512) < 2 ? 2 : (1 << LOG2N) / (CH * 512);
    static constexpr uint32_t TILE = (uint32_t)NW * CH * kChunk;
};

// Geo<m, log2 N, center>::TILE on the host.
inline uint64_t fast_tile(uint32_t m, uint64_t N, bool center) {
    const uint64_t ch = N == 32768 ? 4 : (center && m > 2 && N < 8192 ? 1 : 2);
    return N > 2 * ch * kChunk ? N : 2 * ch * kChunk;
}

// Everything a workgroup needs to know about its worker, in registers; the pointers are uniform.
struct FastCtx {
    float* __restrict__ norms;
    unsigned char* __restrict__ signs;
    unsigned char* __restrict__ levels;
    uint32_t lane, wave, worker, round, key0, key1;
    float smax;
    bool codes_cached;
    unsigned char* string;       // kStringBytes<M> of LDS that are the wave's (level widths 3, 5, 6, 7)
};

// One tile: bucket totals, scales, variates, rounding, packing, stores.  ACC: the dequantised codes are also
// added to acc[chunk][0..8) (the server's sum over workers, for the launch that runs a whole round).
// FULL = false: the ragged last tile of a vector, of which the first `count` coordinates exist and the rest
// of v is 0.
template <int M, int LOG2N, bool ACC = false, class G = Geo<M, LOG2N>, bool FULL = true>
__device__ __forceinline__ void process_tile(const FastCtx& cx, float (&v)[G::CH][8], uint32_t t, float* sm,
                                             float (*acc)[8] = nullptr, uint32_t count = G::TILE) {
    constexpr int CH = G::CH;
    constexpr uint32_t N = 1u << LOG2N;
    constexpr uint32_t TILE = G::TILE;
    constexpr uint32_t LPB = (N < kChunk ? N : kChunk) / kLaneElems;                       // lanes per bucket
    constexpr int CPB = N <= kChunk ? 1 : (int)(N / kChunk < (uint32_t)CH ? N / kChunk : (uint32_t)CH);  // chunks per bucket in a wave
    constexpr uint32_t WPB = N <= CH * kChunk ? 1u : N / (CH * kChunk);                     // waves per bucket
    constexpr int KIND = QESGD_NORM_L2;
    const uint64_t g0 = (uint64_t)t * (TILE / kLaneElems);        // first lane group (8 coordinates) of the tile

    float tot[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) tot[c] = lane_butterfly<KIND>(lane_tree<KIND>(v[c]), LPB);
    if (CPB > 1) {
#pragma unroll
        for (int w = 1; w < CPB; w <<= 1) {
#pragma unroll
            for (int c = 0; c < CH; c += 2 * w) tot[c] = combine<KIND>(tot[c], tot[c + w]);
        }
    }
    if (WPB > 1) {
        if (cx.lane == 0) sm[cx.wave] = tot[0];
        __syncthreads();
        tot[0] = lds_tree16<KIND>(sm, cx.wave & ~(WPB - 1u), WPB);
    }

    Scale sc;
    float step = 0.0f;
    float* __restrict__ norms = cx.norms + (g0 >> (LOG2N - 3));
    unsigned char* __restrict__ signs = cx.signs + g0;
    unsigned char* __restrict__ levels = cx.levels + g0 * M;
    uint32_t sign_byte[CH], bits[CH][4];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const uint32_t idx = (cx.wave * (uint32_t)CH + (uint32_t)c) * kWaveSize + cx.lane;   // lane group inside the tile
        if (c % CPB == 0) {                                       // first chunk of a bucket (or of its part in this wave)
            // a lane beyond the last bucket must not take its wave out of the short rounding: any ordinary scale
            const bool live = FULL || ((idx * kLaneElems) & ~(N - 1u)) < count;
            sc = scale_of_total<M, KIND>(live ? tot[c] : 1.0f);
            if (ACC) step = sc.norm / cx.smax;
            if ((idx & (N / kLaneElems - 1u)) == 0u && live) norms[idx >> (LOG2N - 3)] = sc.norm;
        }
        // the tile starts at a multiple of its size, so the low word of the group number cannot carry
        uint32_t rnd[4];
        philox4x32_10((uint32_t)g0 + idx, (uint32_t)(g0 >> 32), cx.worker, cx.round, cx.key0, cx.key1, rnd);
        round_and_pack<M>(v[c], rnd, sc, sign_byte[c], bits[c]);
        if (ACC) accumulate8<M>(acc[c], sign_byte[c], bits[c], step);
        if (!FULL) {
            const uint32_t rest = count_from(count, idx * kLaneElems);
            store_codes<M>(reinterpret_cast<uint32_t*>(cx.signs), reinterpret_cast<uint32_t*>(cx.levels),
                           (g0 + idx) * kLaneElems, rest < 8u ? rest : 8u, cx.lane, sign_byte[c], bits[c]);
        } else if constexpr (32 % M != 0) {
            store_whole<M>(cx.string, cx.signs, cx.levels, (g0 + idx - cx.lane) * kLaneElems, cx.lane, cx.codes_cached, sign_byte[c], bits[c]);
        }
    }
    if constexpr (FULL && 32 % M == 0)
        store_chunks<M, CH>(signs, levels, cx.wave * (uint32_t)CH * kWaveSize + cx.lane, cx.codes_cached, sign_byte, bits);
}

}  // namespace
}  // namespace qesgd
