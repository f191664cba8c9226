// Worker side of a QESGD round on gfx950: bucket scale, stochastic rounding
// (Sec. 2.1, Eq. (2)) and bit packing, one pass over the input.
//
// Mapping.  The coordinates are laid out in "slot space": bucket b owns the N
// slots [b*N, (b+1)*N), N = bucket size zero-padded to a power of two, so that
// every bucket starts on a power-of-two boundary whatever its length.  A lane
// owns 8 consecutive slots (two 128-bit loads, one Philox call, one sign byte),
// a wavefront owns CH chunks of 64 x 8 = 512 slots, a workgroup owns a tile of
// nwaves x CH x 512 slots.  The fp32 sum of squares is the balanced binary tree
// over slot index bits: bits 0-2 inside the lane, bits 3-8 as an xor butterfly
// over lanes (DPP for masks 1,2,4,8; row / half swaps for 16,32), then the
// chunks of a wave, then the waves of a workgroup through LDS.  Every lane ends
// with its bucket's total, so the scale never goes through memory.
//
// The kernels share the arithmetic:
//   k_quantize_pack_fast  power-of-two buckets, L2 scale, level width dividing 32.  N is a template
//                         parameter, so a tile is straight-line code without guards; the ragged last
//                         tile of a worker runs the same code with masked loads and stores.
//   k_quantize_pack_center  the same with a center and several workers, one tile of every worker.
//   k_quantize_pack_bucket  buckets that are not a power of two, max-norm, level widths 3/5/6/7, and the
//                         last pass of the buckets among them that are too wide for one workgroup.
//   k_quantize_pack_lanes  of those the ones padded to 512 or less, lane by lane.
//   k_tile_partials(_fast), k_finish_norms, k_quantize_pack_pre_fast
//                         buckets wider than kMaxSinglePassBucket: per-tile tree sums into the
//                         workspace, the rest of each bucket's tree, then the quantiser.
#include <mutex>

#include "qesgd_quantize_device.h"

// Scratch of the entry point that allocates nothing: the partial sums of the two-pass path for
// callers that cannot bring a workspace.  One copy per GPU, held until the process ends; every
// call on a GPU shares it.  In host code this name is only a handle for hipGetSymbolAddress.
static __device__ __align__(256) float scratch[qesgd::kStaticScratchFloats];

namespace qesgd {
namespace {

// Worker and tile of a workgroup in the grid of center_grid.  All workers read the same `center`: the K workgroups of one
// tile get ids 8 apart, so they run on one XCD one after the other, and all but the first find the tile of `center` in its L2.
__device__ __forceinline__ void center_order(uint32_t& k, uint32_t& t) {
    k = blockIdx.x >> 3;
    t = (blockIdx.z * gridDim.y + blockIdx.y) * 8u + (blockIdx.x & 7u);
}

// Buckets that the fast kernel does not take but whose coordinates a wave finds side by side: the max norm, level widths
// 3, 5, 6 and 7, sizes that are no power of two.  What depends on the size is scalar work, so one kernel serves all sizes.
//   kBuckets  padded to 1024 .. 32768: a bucket is a few waves, whose totals meet in LDS; a workgroup holds whole buckets
//   kNarrow   up to 512, a power of two or the only one: slot == coordinate, several buckets in a wave
//   kPre      last pass of buckets wider than kMaxSinglePassBucket: the scale is read from the norms plane
// A wave is whole, ragged, or all padding (then it only meets the others); only a ragged one guards its lanes.
// Bound by vector issue (d = 7.3 M, K = 5, s = 32, bucket 3008, max norm: 339 vector instructions per 1024 coordinates,
// 428 and 1.5 times the scalar ones where every wave guarded itself).  Guarded / this, quantiser alone:
//   d = 7.3 M, K = 5, s = 32, bucket 3008, max    48.5 -> 40.7 us
//   d = 20 M, K = 8, s = 4, bucket 2400, max      174 -> 141 us
//   d = 15 M, K = 5, s = 4, bucket 23648, max     84.7 -> 60.0 us
//   d = 30 M, K = 8, s = 64, bucket 32768         271 -> 214 us
// With a center the workers of a tile follow one another (center_order); quantiser, all tiles of a worker first / this:
//   d = 60 M, K = 8, s = 16, bucket 992           577 -> 478 us
//   d = 60 M, K = 8, s = 16, bucket 12000         548 -> 534 us
//   d = 60 M, K = 8, s = 16, bucket 224           773 -> 497 us (lane by lane)
enum Mode { kBuckets, kNarrow, kPre };
template <int M, int CH, int KIND, bool CENTER, Mode MODE>
__device__ __forceinline__ void pack_bucket(const QParams& p) {
    __shared__ float sm[16];
    extern __shared__ __align__(16) unsigned char strings[];
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t k = blockIdx.y, t = blockIdx.x;
    if (CENTER) {
        center_order(k, t);
        if (t >= p.full_tiles) return;
    }
    const uint64_t unit = ((uint64_t)xcd_tile(t, CENTER ? p.full_tiles : gridDim.x, p.xcd_group) << p.log2_waves) + wave;
    const uint32_t lg = p.log2N - (CH == 4 ? 11u : 10u);                         // log2 of a bucket's waves
    static_assert(CH == 2 || CH == 4, "");
    const WaveSpan s = MODE == kNarrow ? wave_span_dense<CH>(p, unit) : wave_span<CH>(p, unit, lg);
    float v[CH][8];
    load_span<CH, CENTER>(p, k, s, lane, v);
    float* __restrict__ norms = reinterpret_cast<float*>(p.packed + (uint64_t)k * p.packed_stride + p.norms_off);

    Scale sc[CH];
    if (MODE == kPre) {
        if (s.mine == 0) return;
        sc[0] = scale_of_norm<M>(norms[s.bucket]);
    } else {
        const uint32_t lanes = MODE == kNarrow ? 1u << (p.log2N - 3u) : 64u;     // that share a bucket
        float tot[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) tot[c] = lane_butterfly<KIND>(lane_tree<KIND>(v[c]), lanes);
        if (MODE == kNarrow) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                // a lane beyond the last bucket must not take its wave out of the short rounding: any ordinary scale
                const uint32_t at = (uint32_t)c * kChunk + lane * kLaneElems;
                const bool live = (at & ~(lanes * kLaneElems - 1u)) < s.mine;
                sc[c] = scale_of_total<M, KIND>(live ? tot[c] : 1.0f);
                if ((lane & (lanes - 1u)) == 0u && live) norms[(s.i0 + at) >> p.log2N] = sc[c].norm;
            }
        } else {
#pragma unroll
            for (int w = 1; w < CH; w <<= 1)
#pragma unroll
                for (int c = 0; c < CH; c += 2 * w) tot[c] = combine<KIND>(tot[c], tot[c + w]);
            if (lg > 0) {                                                        // the same for the workgroup
                const uint32_t waves = 1u << lg;
                if (lane == 0) sm[wave] = tot[0];
                __syncthreads();
                tot[0] = lane_butterfly<KIND>(sm[(wave & ~(waves - 1u)) + (lane & (waves - 1u))], waves);
            }
            if (s.mine == 0) return;
            sc[0] = scale_of_total<M, KIND>(tot[0]);
            if (s.sub == 0 && lane == 0) norms[s.bucket] = sc[0].norm;
        }
    }
    if (MODE != kNarrow) {
#pragma unroll
        for (int c = 1; c < CH; ++c) sc[c] = sc[0];
    }
    encode_span<M, CH, KIND>(p, k, s, lane, strings + wave * kStringBytes<M>, v, sc);
}
// Two workgroups of 16 waves fit a CU if a wave has at most 96 scalar registers, of which the trap handler holds 16.  The
// compiler counts without those and takes 82 for levels of 7 bits, with which one fits; their buckets padded to 16384 have a
// kernel of their own that is held to 80 (quantiser, d = 25.6 M, K = 4, s = 128, bucket 16384 111 -> 89 us).  Smaller workgroups lose
// by the limit (d = 3.5 M, K = 8, s = 128, bucket 992, max norm 27.3 -> 29.8 us).
template <int M, int CH>
constexpr bool kOwn16 = M == 7 && CH == 2;
template <int M, int CH, int KIND, bool CENTER, Mode MODE>
__global__ void __launch_bounds__((MODE != kBuckets ? 256 : kOwn16<M, CH> ? 512 : 1024)) k_quantize_pack_bucket(const QParams p) {
    pack_bucket<M, CH, KIND, CENTER, MODE>(p);
}
template <int M, int KIND, bool CENTER>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_num_sgpr(80))) k_quantize_pack_bucket16(const QParams p) {
    pack_bucket<M, 2, KIND, CENTER, kBuckets>(p);
}

// The buckets that neither takes (see LaneSpan).  (Through whole-line loads and an exchange: d = 15 M, K = 5, s = 16,
// bucket 320 84.0 us, lane by lane 76.0.)
template <int M, int KIND, bool CENTER>
__global__ void __launch_bounds__(256) k_quantize_pack_lanes(const QParams p) {
    constexpr int CH = 2;
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t N = 1ull << p.log2N;
    uint32_t k = blockIdx.y, t = blockIdx.x;
    if (CENTER) {
        center_order(k, t);
        if (t >= p.full_tiles) return;
    }
    const uint64_t slot0 = ((uint64_t)xcd_tile(t, CENTER ? p.full_tiles : gridDim.x, p.xcd_group) * 4u + (threadIdx.x >> 6)) * (CH * kChunk);
    LaneSpan span[CH];
    float v[CH][8];
#pragma unroll
    for (int c = 0; c < CH; ++c) span[c] = lane_span(slot0 + (uint32_t)c * kChunk + lane * kLaneElems, p);
    load_lanes<CH, CENTER>(p, k, span, v);
    unsigned char* __restrict__ out = p.packed + (uint64_t)k * p.packed_stride;
    float* __restrict__ norms = reinterpret_cast<float*>(out + p.norms_off);
    Scale scale[CH];                                      // of all chunks before the first store
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const float tot = lane_butterfly<KIND>(lane_tree<KIND>(v[c]), (uint32_t)(N / kLaneElems));
        scale[c] = scale_of_total<M, KIND>(span[c].nvalid || N == kChunk ? tot : 1.0f);      // (see kNarrow)
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        Scale sc = scale[c];
        if (span[c].opens_bucket) norms[span[c].bucket] = sc.norm;
        // a chunk opens a bucket: if that holds no coordinate, the vector has ended
        if (__builtin_amdgcn_readfirstlane(span[c].nvalid) == 0u) continue;
        const uint64_t g = span[c].i / kLaneElems;
        uint32_t rnd[4], sign_byte, bits[4];
        philox4x32_10((uint32_t)g, (uint32_t)(g >> 32), p.worker0 + k, p.round, p.key0, p.key1, rnd);
        if (KIND != QESGD_NORM_L2) sc.direct = sc.direct && wave_all(no_nan<KIND>(v[c]));
        round_and_pack<M>(v[c], rnd, sc, sign_byte, bits);
        store_codes<M>(reinterpret_cast<uint32_t*>(out + p.signs_off), reinterpret_cast<uint32_t*>(out + p.levels_off), span[c].i,
                       span[c].nvalid, lane, sign_byte, bits);
    }
}

// At most six waves per SIMD for the kernels that stream whole tiles, where it pays: their registers would allow eight, which
// are more streams than the memory takes at full rate.  The launch says so by the LDS that it asks for (six_wave_lds).
// Quantiser, eight / six waves, two inputs in turn, us; MB of the vectors + the codes:
//   up to 4 waves per workgroup, from 320 MiB or 48 MiB of codes on
//                  s = 2, 4096, 4222 + 263 MB 814 / 793;  s = 4, 2048, 1831 + 171 340 / 329;  s = 16, 512, 1559 + 243 415 / 398
//                  s = 256, 2048, 183 + 51 38.3 / 37.6;  s = 2, 2048, 457 + 28 80.1 / 78.3;  s = 65536, 128, 97 + 51 26.8 / 26.3
//                  but s = 2, 512, 97 + 6 17.8 / 18.7, 183 + 11 32.5 / 33.9, 366 + 22 64.2 / 64.7;  s = 16, 512, 122 + 19 25.0 / 25.6
//   8 waves (8192), whose barrier wants more of them, where the codes go out non-temporally
//                  s = 256, 1559 + 438 331 / 309, 779 + 219 166 / 156;  s = 4, 1831 + 171 334 / 336;  but s = 16, 779 + 121 146 / 153
//   one bucket     s = 256, 1559 + 438 MB 551 / 533 (both passes; only the second one 536)
//   with a center  one worker, s = 256, 2048, 527 + 148 MB 2% faster, or up to 2 bits, K = 2, s = 2, 2048, 457 + 28 131 / 128;
//                  but K = 4, s = 256, 4096, 183 + 51 44.7 / 49.3
// A workgroup of 16 waves is alone on a CU or one of two, four or eight waves per SIMD: four lose (bucket 16384, d = 138 M, K = 8,
// s = 2 819 / 983).  k_quantize_pack_center is indifferent (d = 57 M, K = 4, s = 16, bucket 4096 232 / 231), the general kernels need
// the waves (d = 20 M, K = 8, s = 4, bucket 2400, max norm 134 / 147).

// One tile per workgroup.  (Walking several tiles per workgroup with the next tile's loads in flight was
// measured and is slower: the packed stores of a long-lived workgroup spread out in time and the mixed
// read/write stream to HBM loses more than the prefetch gains.)
// Bound by the mix of reads and writes: at d = 138 M, K = 8, s = 2, bucket 4096, with eight waves per SIMD, it took 811 us,
// 610 us with the stores left out (7.3 TB/s) and 813 us without Philox.  Before (32 bytes per lane, ordinary policy, general
// rounding, tiles dealt round-robin) / with eight waves / with six, two inputs in turn:
//   d = 138 M, K = 8, s = 2, bucket 4096     850 / 811 / 793 us = 5.9 TB/s
//   d = 25.6 M, K = 16, s = 256, bucket 8192 380 / 331 / 309 us = 6.8 TB/s
//   d = 60 M, K = 8, s = 4, bucket 2048      364 / 340 / 329 us = 6.4 TB/s
template <int M, int LOG2N, bool CENTER>
__global__ void __launch_bounds__((Geo<M, LOG2N, CENTER>::NW * 64)) k_quantize_pack_fast(const QParams p) {
    constexpr int CH = Geo<M, LOG2N, CENTER>::CH;
    constexpr uint32_t TILE = Geo<M, LOG2N, CENTER>::TILE;
    __shared__ float sm[32];

    // Grid: (tiles, workers), so that nothing has to be divided; with a center (8 * workers, y, z).
    const uint32_t tiles = p.full_tiles + p.tail_tiles;
    uint32_t k = blockIdx.y, t = blockIdx.x;
    if (CENTER) {
        center_order(k, t);
        if (t >= tiles) return;
    }
    t = xcd_tile(t, tiles, p.xcd_group);
    const float* __restrict__ xk = p.x + (uint64_t)k * p.x_stride;
    const float* __restrict__ ck = p.center;
    unsigned char* __restrict__ out = p.packed + (uint64_t)k * p.packed_stride;
    FastCtx cx;
    cx.norms = reinterpret_cast<float*>(out + p.norms_off);
    cx.signs = out + p.signs_off;
    cx.levels = out + p.levels_off;
    cx.lane = threadIdx.x & 63u;
    cx.wave = threadIdx.x >> 6;
    cx.worker = p.worker0 + k;
    cx.round = p.round;
    cx.key0 = p.key0;
    cx.key1 = p.key1;
    cx.smax = p.smax;
    cx.codes_cached = p.codes_cached;

    float buf[CH][8];
    const uint64_t w0 = (uint64_t)t * TILE + cx.wave * (uint32_t)(CH * kChunk);
    if (t >= p.full_tiles) {                              // the ragged last tile of the worker (at most one)
        const uint32_t count = (uint32_t)(p.d - (uint64_t)t * TILE);
        load_tile<CH, CENTER, false>(xk + w0, ck + w0, cx.lane, true, buf, count_from(count, cx.wave * (uint32_t)(CH * kChunk)));
        process_tile<M, LOG2N, false, Geo<M, LOG2N, CENTER>, false>(cx, buf, t, sm, nullptr, count);
        return;
    }
    load_tile<CH, CENTER>(xk + w0, ck + w0, cx.lane, p.x_cached, buf);
    process_tile<M, LOG2N, false, Geo<M, LOG2N, CENTER>>(cx, buf, t, sm);
}

// The center form for several workers: a workgroup owns one tile of every worker, keeps the tile
// of `center` in registers and takes the workers one after the other with the next worker's loads
// in flight, so `center` is read once per tile instead of once per tile and worker.  Buckets of 32768 spill (200 to
// 272 bytes per lane at the 128 registers that 1024 threads leave).
template <int M, int LOG2N>
__global__ void __launch_bounds__((Geo<M, LOG2N, true>::NW * 64)) k_quantize_pack_center(const QParams p) {
    constexpr int CH = Geo<M, LOG2N, true>::CH;
    constexpr uint32_t TILE = Geo<M, LOG2N, true>::TILE;
    __shared__ float sm[2][32];             // alternate per worker: one barrier per tile suffices
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x, p.xcd_group);
    const uint32_t K = p.group_workers;
    FastCtx cx;
    cx.lane = threadIdx.x & 63u;
    cx.wave = threadIdx.x >> 6;
    cx.round = p.round;
    cx.key0 = p.key0;
    cx.key1 = p.key1;
    cx.smax = p.smax;
    cx.codes_cached = p.codes_cached;
    const uint64_t e0 = (uint64_t)t * TILE;
    if (t >= p.full_tiles) {                              // the ragged last tile
        const uint32_t count = (uint32_t)(p.d - e0), first = cx.wave * (uint32_t)(CH * kChunk);
        for (uint32_t k = 0; k < K; ++k) {
            unsigned char* __restrict__ out = p.packed + (uint64_t)k * p.packed_stride;
            cx.norms = reinterpret_cast<float*>(out + p.norms_off);
            cx.signs = out + p.signs_off;
            cx.levels = out + p.levels_off;
            cx.worker = p.worker0 + k;
            float v[CH][8];
            load_tile<CH, true, false>(p.x + (uint64_t)k * p.x_stride + e0 + first, p.center + e0 + first, cx.lane, true, v,
                                       count_from(count, first));
            process_tile<M, LOG2N, false, Geo<M, LOG2N, true>, false>(cx, v, t, sm[k & 1u], nullptr, count);
        }
        return;
    }
    const uint64_t w0 = e0 + cx.wave * (uint32_t)(CH * kChunk) + half_offset(cx.lane);
    vec4 ca[CH], cb[CH], a[CH], b[CH], na[CH], nb2[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const uint64_t o = w0 + (uint32_t)c * kChunk;
        ca[c] = load_stream(p.center + o);
        cb[c] = load_stream(p.center + o + kChunk / 2);
        a[c] = load_stream(p.x + o);
        b[c] = load_stream(p.x + o + kChunk / 2);
    }
    for (uint32_t k = 0; k < K; ++k) {
        if (k + 1 < K) {
            const float* __restrict__ xn = p.x + (uint64_t)(k + 1) * p.x_stride + w0;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                na[c] = load_stream(xn + (uint32_t)c * kChunk);
                nb2[c] = load_stream(xn + (uint32_t)c * kChunk + kChunk / 2);
            }
        }
        float v[CH][8];
#pragma unroll
        for (int c = 0; c < CH; ++c) halves_to_lane(a[c] - ca[c], b[c] - cb[c], v[c]);
        unsigned char* __restrict__ out = p.packed + (uint64_t)k * p.packed_stride;
        cx.norms = reinterpret_cast<float*>(out + p.norms_off);
        cx.signs = out + p.signs_off;
        cx.levels = out + p.levels_off;
        cx.worker = p.worker0 + k;
        process_tile<M, LOG2N, false, Geo<M, LOG2N, true>>(cx, v, t, sm[k & 1u]);
        if (k + 1 < K) {
#pragma unroll
            for (int c = 0; c < CH; ++c) { a[c] = na[c]; b[c] = nb2[c]; }
        }
    }
}

// Tree sum (or max) of one 4096-slot tile of worker k, left in the workspace.  Tiles of a bucket are consecutive in
// slot space, so the workspace index of (bucket, tile in bucket) is the tile index.  sm: 4 floats of LDS.
template <int KIND, bool CENTER>
__device__ __forceinline__ void partial_tile(const QParams& p, uint32_t k, uint32_t tile, float* sm) {
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const WaveSpan s = wave_span<2>(p, (uint64_t)tile * 4u + wave, p.log2N - 10u);
    float v[2][8];
    load_span<2, CENTER>(p, k, s, lane, v);
    const float t = combine<KIND>(lane_butterfly<KIND>(lane_tree<KIND>(v[0]), 64), lane_butterfly<KIND>(lane_tree<KIND>(v[1]), 64));
    if (lane == 0) sm[wave] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float total = combine<KIND>(combine<KIND>(sm[0], sm[1]), combine<KIND>(sm[2], sm[3]));
        p.workspace[(uint64_t)k * p.ws_tiles_per_worker + tile] = total;
    }
}

// Buckets wider than kMaxSinglePassBucket, tiles wholly inside the vector (slot == coordinate:
// power-of-two bucket, or a single bucket).  First pass: tree sum of one 4096-coordinate tile into
// the workspace.  Last pass: the quantiser with the bucket scale read from the norms plane; a tile
// never straddles two such buckets, so the scale is one scalar per workgroup.
// Both walk (tiles, workers) in the same order, so that a vector that fits the L2s is found in the same one.
template <bool CENTER>
__global__ void __launch_bounds__(256) k_tile_partials_fast(const QParams p) {
    constexpr int KIND = QESGD_NORM_L2;
    __shared__ float sm[4];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t k = blockIdx.y;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x, p.xcd_group);
    if (t >= p.full_tiles) {                              // the ragged last tile of the worker (at most one)
        partial_tile<KIND, CENTER>(p, k, t, sm);
        return;
    }
    const uint64_t w0 = (uint64_t)t * kPartialTile + wave * (2u * kChunk);
    float v[2][8];
    load_tile<2, CENTER>(p.x + (uint64_t)k * p.x_stride + w0, p.center + w0, lane, p.x_cached, v);
    const float t0 = lane_butterfly<KIND>(lane_tree<KIND>(v[0]), 64);
    const float t1 = lane_butterfly<KIND>(lane_tree<KIND>(v[1]), 64);
    if (lane == 0) sm[wave] = t0 + t1;
    __syncthreads();
    if (threadIdx.x == 0) p.workspace[(uint64_t)k * p.ws_tiles_per_worker + t] = (sm[0] + sm[1]) + (sm[2] + sm[3]);
}

// merged: every wave finishes its bucket's tree by itself while its coordinates are on their way, which
// saves the launch between the passes; the bucket's first tile writes the scale.
template <int M, bool CENTER>
__global__ void __launch_bounds__(256) k_quantize_pack_pre_fast(const QParams p) {
    __shared__ __align__(16) unsigned char strings[4][kStringBytes<M> + 16];
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t k = blockIdx.y;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x, p.xcd_group);
    unsigned char* __restrict__ out = p.packed + (uint64_t)k * p.packed_stride;
    float* __restrict__ norms = reinterpret_cast<float*>(out + p.norms_off);
    const uint64_t b = (uint64_t)t * kPartialTile >> p.log2N;
    const bool full = t < p.full_tiles;                   // one condition for the workgroup, no other for its waves
    const uint64_t w0 = (uint64_t)t * kPartialTile + wave * (2u * kChunk);
    WaveSpan s{};
    float v[2][8];
    if (full) {
        load_tile<2, CENTER>(p.x + (uint64_t)k * p.x_stride + w0, p.center + w0, lane, p.x_cached, v);
    } else {                                              // the ragged last tile of the worker (at most one)
        s = wave_span_dense<2>(p, (uint64_t)t * 4u + wave);
        load_span<2, CENTER>(p, k, s, lane, v);
    }
    Scale sc;
    if (p.merged) {
        const uint32_t P = 1u << (p.log2N - 12u);
        const uint64_t left = p.data_tiles - b * P;
        const float* __restrict__ ws = p.workspace + (uint64_t)k * p.ws_tiles_per_worker + b * P;
        sc = scale_of_total<M, QESGD_NORM_L2>(wave_total<QESGD_NORM_L2>(ws, P, left < P ? (uint32_t)left : P, lane));
        if (threadIdx.x == 0 && (t & (P - 1u)) == 0u) norms[b] = sc.norm;
    } else {
        sc = scale_of_norm<M>(norms[b]);
    }
    const Scale both[2] = {sc, sc};
    if (full) encode_whole<M, 2, QESGD_NORM_L2>(p, k, w0, lane, strings[wave], v, both);
    else encode_span<M, 2, QESGD_NORM_L2>(p, k, s, lane, strings[wave], v, both);
}

// ---------------------------------------------------------------------------
// Buckets wider than kMaxSinglePassBucket that are no power of two, and the max norm: pass A leaves
// the tree sum of a 4096-slot tile in the workspace, pass B finishes the tree per bucket and writes
// the scale, then k_quantize_pack_bucket<.., kPre> reads it.
// workspace[(k*nb + b)*P + t], P = N / 4096.
// ---------------------------------------------------------------------------
template <int KIND, bool CENTER>
__global__ void k_tile_partials(const QParams p) {
    __shared__ float sm[4];
    partial_tile<KIND, CENTER>(p, blockIdx.y, xcd_tile(blockIdx.x, gridDim.x, p.xcd_group), sm);
}

// Finishes the tree of one bucket: P leaves (a power of two, >= 16), of which only the first
// `valid` were written (the rest of the padded bucket is +0, the identity of both combines, and is
// never read).  One workgroup of W = 1..16 waves per (worker, bucket) walks the leaves in tiles of
// W x 2 chunks x 512, each reduced like a tile of the first pass (leaf index bits 0-2 in the
// lane, 3-8 across lanes, 9 across the two chunks, then the waves); the tile totals are joined by
// a binary counter: stack[l] holds the finished subtree of 2^l tiles that waits for its right
// sibling.  W is the largest power of two with W x 1024 <= max(P, 1024).
template <int KIND>
__global__ void __launch_bounds__(1024) k_finish_norms(const QParams p, uint64_t P, uint32_t dense) {
    __shared__ float sm[2][16];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t nwaves = blockDim.x >> 6;
    const uint64_t tile = (uint64_t)nwaves * 1024u;
    const uint64_t kb = blockIdx.x;                     // k*nb + b
    const uint32_t k = (uint32_t)(kb / p.nb);
    const uint64_t b = kb - (uint64_t)k * p.nb;
    const float* __restrict__ ws = p.workspace + kb * P;
    uint64_t valid = P;
    if (dense) {
        const uint64_t left = p.data_tiles - b * P;     // buckets before the last are full
        valid = left < P ? left : P;
    }
    const uint64_t iters = (P + tile - 1) / tile;                         // a power of two
    float stack[16];
#pragma unroll
    for (int l = 0; l < 16; ++l) stack[l] = 0.0f;
    for (uint64_t it = 0; it < iters; ++it) {
        float total = 0.0f;
        const uint64_t base = it * tile;
        if (base < valid) {                              // uniform: tiles beyond `valid` are all +0
            float t2[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint64_t j = base + wave * 1024u + (uint32_t)c * kChunk + lane * kLaneElems;
                float q[8];
                if (j + 8 <= valid) {
                    const float4 a0 = *reinterpret_cast<const float4*>(ws + j);
                    const float4 a1 = *reinterpret_cast<const float4*>(ws + j + 4);
                    q[0] = a0.x; q[1] = a0.y; q[2] = a0.z; q[3] = a0.w;
                    q[4] = a1.x; q[5] = a1.y; q[6] = a1.z; q[7] = a1.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) q[e] = (j + e < valid) ? ws[j + e] : 0.0f;
                }
                t2[c] = lane_butterfly<KIND>(lane_tree_of_partials<KIND>(q), 64);
            }
            float* buf = sm[it & 1u];
            if (lane == 0) buf[wave] = combine<KIND>(t2[0], t2[1]);
            __syncthreads();                             // one barrier per tile: the buffers alternate
            total = lds_tree16<KIND>(buf, 0, nwaves);
        }
#pragma unroll
        for (int l = 0; l < 16; ++l) {                   // 16 waves whenever P > 16384: iters <= 2^40 / 4096 / 16384 = 2^14
            if (((it >> l) & 1u) == 0u) { stack[l] = total; break; }
            total = combine<KIND>(stack[l], total);
        }
    }
    if (threadIdx.x == 0) {
        float result = stack[0];
#pragma unroll
        for (int l = 1; l < 16; ++l)
            if ((iters >> l) & 1u) result = stack[l];
        float* norms = reinterpret_cast<float*>(p.packed + (uint64_t)k * p.packed_stride + p.norms_off);
        norms[b] = (KIND == QESGD_NORM_L2) ? sqrtf(result) : result;
    }
}

// ---------------------------------------------------------------------------
// Launch plumbing.
// ---------------------------------------------------------------------------
dim3 center_grid(uint32_t tiles, uint32_t workers) {
    const uint32_t octets = (tiles + 7u) / 8u, gz = (octets + 65534u) / 65535u, gy = (octets + gz - 1u) / gz;
    return dim3(8u * workers, gy, gz);
}

// CH, MODE: of k_quantize_pack_bucket; CH = 0: k_quantize_pack_lanes.
template <int M, int CH, Mode MODE, int KIND, bool CENTER>
void launch_general_one(const QParams& p, dim3 grid, dim3 block, hipStream_t st) {
    if (CENTER) grid = center_grid(grid.x, grid.y);
    const uint32_t lds = (block.x >> 6) * kStringBytes<M>;
    if constexpr (CH == 0) {
        hipLaunchKernelGGL((k_quantize_pack_lanes<M, KIND, CENTER>), grid, block, 0, st, p);
    } else {
        if constexpr (MODE == kBuckets && kOwn16<M, CH>) {
            if (block.x == 1024) {
                hipLaunchKernelGGL((k_quantize_pack_bucket16<M, KIND, CENTER>), grid, block, lds, st, p);
                return;
            }
        }
        hipLaunchKernelGGL((k_quantize_pack_bucket<M, CH, KIND, CENTER, MODE>), grid, block, lds, st, p);
    }
}

template <int M, int CH, Mode MODE>
void launch_general_m(const QParams& p, uint32_t norm_kind, dim3 grid, dim3 block, hipStream_t st) {
    if (norm_kind == QESGD_NORM_L2) {
        if (p.center) launch_general_one<M, CH, MODE, QESGD_NORM_L2, true>(p, grid, block, st);
        else launch_general_one<M, CH, MODE, QESGD_NORM_L2, false>(p, grid, block, st);
    } else {
        if (p.center) launch_general_one<M, CH, MODE, QESGD_NORM_MAX, true>(p, grid, block, st);
        else launch_general_one<M, CH, MODE, QESGD_NORM_MAX, false>(p, grid, block, st);
    }
}

template <int CH, Mode MODE>
void launch_general(const QParams& p, uint32_t m, uint32_t norm_kind, dim3 grid, dim3 block, hipStream_t st) {
    switch (m) {
        case 1: launch_general_m<1, CH, MODE>(p, norm_kind, grid, block, st); break;
        case 2: launch_general_m<2, CH, MODE>(p, norm_kind, grid, block, st); break;
        case 3: launch_general_m<3, CH, MODE>(p, norm_kind, grid, block, st); break;
        case 4: launch_general_m<4, CH, MODE>(p, norm_kind, grid, block, st); break;
        case 5: launch_general_m<5, CH, MODE>(p, norm_kind, grid, block, st); break;
        case 6: launch_general_m<6, CH, MODE>(p, norm_kind, grid, block, st); break;
        case 7: launch_general_m<7, CH, MODE>(p, norm_kind, grid, block, st); break;
        case 8: launch_general_m<8, CH, MODE>(p, norm_kind, grid, block, st); break;
        default: launch_general_m<16, CH, MODE>(p, norm_kind, grid, block, st); break;
    }
}

template <int KIND>
void launch_partials(const QParams& p, dim3 grid, hipStream_t st) {
    if (p.center) hipLaunchKernelGGL((k_tile_partials<KIND, true>), grid, dim3(256), 0, st, p);
    else hipLaunchKernelGGL((k_tile_partials<KIND, false>), grid, dim3(256), 0, st, p);
}

// Dynamic LDS of a kernel that streams whole tiles (see k_quantize_pack_fast); fixed: what it has besides.
uint32_t stream_lds(const QParams& p, uint32_t waves, uint32_t fixed) {
    return p.six_waves && (waves < 8u || !p.codes_cached) ? six_wave_lds(waves, fixed) : 0u;
}
constexpr uint32_t kFastLds = 128;

template <int M, int LOG2N>
void launch_fast_one(const QParams& p, hipStream_t st) {
    const uint32_t tiles = p.full_tiles + p.tail_tiles;
    // With a center and enough tiles to fill the chip many times over (measured: it pays from about
    // 64 waves per SIMD on), a workgroup takes one tile of every worker and reads `center` once.
    if (p.center && p.group_workers > 1 && (uint64_t)p.full_tiles * Geo<M, LOG2N, true>::NW >= 65536u) {
        hipLaunchKernelGGL((k_quantize_pack_center<M, LOG2N>), dim3(tiles), dim3((Geo<M, LOG2N, true>::NW * 64)), 0, st, p);
        return;
    }
    if (p.center) {
        hipLaunchKernelGGL((k_quantize_pack_fast<M, LOG2N, true>), center_grid(tiles, p.group_workers),
                           dim3((Geo<M, LOG2N, true>::NW * 64)), stream_lds(p, Geo<M, LOG2N, true>::NW, kFastLds), st, p);
        return;
    }
    hipLaunchKernelGGL((k_quantize_pack_fast<M, LOG2N, false>), dim3(tiles, p.group_workers),
                       dim3((Geo<M, LOG2N>::NW * 64)), stream_lds(p, Geo<M, LOG2N>::NW, kFastLds), st, p);
}

template <int M>
void launch_fast_n(const QParams& p, hipStream_t st) {
    switch (p.log2N) {
        case 5: launch_fast_one<M, 5>(p, st); break;
        case 6: launch_fast_one<M, 6>(p, st); break;
        case 7: launch_fast_one<M, 7>(p, st); break;
        case 8: launch_fast_one<M, 8>(p, st); break;
        case 9: launch_fast_one<M, 9>(p, st); break;
        case 10: launch_fast_one<M, 10>(p, st); break;
        case 11: launch_fast_one<M, 11>(p, st); break;
        case 12: launch_fast_one<M, 12>(p, st); break;
        case 13: launch_fast_one<M, 13>(p, st); break;
        case 14: launch_fast_one<M, 14>(p, st); break;
        default: launch_fast_one<M, 15>(p, st); break;
    }
}

void launch_fast(const QParams& p, uint32_t m, hipStream_t st) {
    switch (m) {
        case 1: launch_fast_n<1>(p, st); break;
        case 2: launch_fast_n<2>(p, st); break;
        case 4: launch_fast_n<4>(p, st); break;
        case 8: launch_fast_n<8>(p, st); break;
        default: launch_fast_n<16>(p, st); break;
    }
}

template <int M>
void launch_pre_fast_m(const QParams& p, dim3 blocks, hipStream_t st) {
    const uint32_t lds = stream_lds(p, 4, 4u * (kStringBytes<M> + 16u));
    if (p.center) hipLaunchKernelGGL((k_quantize_pack_pre_fast<M, true>), blocks, dim3(256), lds, st, p);
    else hipLaunchKernelGGL((k_quantize_pack_pre_fast<M, false>), blocks, dim3(256), lds, st, p);
}

void launch_pre_fast(const QParams& p, uint32_t m, dim3 blocks, hipStream_t st) {
    switch (m) {
        case 1: launch_pre_fast_m<1>(p, blocks, st); break;
        case 2: launch_pre_fast_m<2>(p, blocks, st); break;
        case 3: launch_pre_fast_m<3>(p, blocks, st); break;
        case 4: launch_pre_fast_m<4>(p, blocks, st); break;
        case 5: launch_pre_fast_m<5>(p, blocks, st); break;
        case 6: launch_pre_fast_m<6>(p, blocks, st); break;
        case 7: launch_pre_fast_m<7>(p, blocks, st); break;
        case 8: launch_pre_fast_m<8>(p, blocks, st); break;
        default: launch_pre_fast_m<16>(p, blocks, st); break;
    }
}

int check_launch() {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_last_hip_error((int)e);
        return QESGD_ERR_HIP;
    }
    return QESGD_OK;
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
float* g_scratch_ptr[kMaxDevices] = {};     // device address of `scratch` on each GPU, looked up once

}  // namespace

// Device address of the current GPU's copy of `scratch`.  The first call on a device asks the
// runtime for the address (each GPU holds its own copy at its own address); later calls read
// the table.
int static_scratch(float** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess && (dev < 0 || dev >= kMaxDevices)) e = hipErrorInvalidDevice;
    if (e != hipSuccess) {
        set_last_hip_error((int)e);
        return QESGD_ERR_HIP;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            set_last_hip_error((int)(e != hipSuccess ? e : hipErrorInvalidSymbol));
            return QESGD_ERR_HIP;
        }
        g_scratch_ptr[dev] = static_cast<float*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return QESGD_OK;
}

QParams quantize_params(const Shape& sh, const QuantizeArgs& a) {
    QParams p{};
    p.x = a.x;
    p.center = a.center;
    p.packed = a.packed;
    p.workspace = a.workspace;
    p.x_stride = a.x_stride;
    p.packed_stride = a.packed_stride;
    p.d = sh.d;
    p.B = sh.B;
    p.nb = sh.nb;
    p.norms_off = sh.lay.norms_off;
    p.signs_off = sh.lay.signs_off;
    p.levels_off = sh.lay.levels_off;
    p.log2N = sh.log2N;
    p.log2_waves = 2;
    p.key0 = (uint32_t)a.seed;
    p.key1 = (uint32_t)(a.seed >> 32);
    p.round = a.round;
    p.worker0 = a.worker0;
    p.smax = (float)(sh.s - 1);
    p.group_workers = a.K;
    p.x_cached = input_cached(sh, a.K);
    p.codes_cached = a.K * sh.lay.payload_bytes <= kCachedCodeBytes;
    p.six_waves = !p.x_cached && (!p.center || a.K == 1 || sh.m <= 2) &&
                  (4u * (uint64_t)a.K * sh.d >= kSixWaveInput || a.K * sh.lay.payload_bytes >= kSixWaveCodes);
    // The ragged waves of buckets that are no power of two are up to all of the input.  They keep the ordinary policy where
    // they fit the memory-side cache next to what else is read again, the codes and the center; beyond that their stream drives
    // those out.  Quantiser, K = 8, ordinary / non-temporal, us; MB of the ragged waves, the codes and the center:
    //   s = 16, bucket 992     3.5 M (129 MB) 20.9 / 22.3, 5 M (185) 33.9 / 30.4
    //   s = 16, bucket 1504    6.5 M (98) 34.6 / 39.6, 10 M (152) 58.7 / 59.4, 13 M (198) 84.2 / 76.5
    //   s = 256, bucket 2016   5 M (124) 30.4 / 33.1, 6.5 M (160) 42.9 / 42.1, 10 M (248) 71.3 / 63.4
    //   s = 256, bucket 12000  10 M (110) 71.7 / 73.5, 13 M (142) 96.3 / 94.1; with a center 8 M (120) 72.3 / 72.4
    //   center, s = 16, 1504   5 M (104) 32.8 / 38.0, 8 M (154) 60.5 / 59.8, 60 M (890) 678 / 573
    // With codes that go out non-temporally, no center and a ragged wave behind each one to three whole ones the ordinary
    // policy is better at any size (K = 16, d = 25.6 M, s = 256, bucket 2016 351 / 396, 3008 350 / 381; K = 8, d = 60 M, s = 16,
    // 2016 379 / 417; but 5024 370 / 372, 992 392 / 375); in buckets wider than 32768, read twice, the other is (K = 16,
    // d = 25.6 M, s = 32, bucket 48000 640 / 575).
    const uint64_t wave = (sh.N == 32768 ? 4u : 2u) * (uint64_t)kChunk;
    const uint64_t kept = 4u * (uint64_t)a.K * sh.nb * (sh.B % wave) + (p.codes_cached ? a.K * sh.lay.payload_bytes : 0u) + (p.center ? 4u * sh.d : 0u);
    p.ragged_cached = p.x_cached || (sh.N <= kMaxSinglePassBucket && kept <= kCachedRaggedBytes) ||
                      (!p.center && !p.codes_cached && sh.N > 2 * kChunk && sh.N <= 4096);
    return p;
}

// First part of the dense two-pass path (slot space equals coordinate space: the bucket is a power of two or
// there is one bucket; L2 scale): partial sums of all workers, and their trees where the last pass does not
// finish them itself.  Up to 512 partial sums per bucket it does: reading them again in every wave then costs
// less than the launch (quantise and aggregate, d = 0.1 M, K = 4, one bucket: 17.6 us with the launch, 14.8
// without; at 25.6 M coordinates every wave would read 25 KB).
constexpr uint64_t kMergePartials = 512;
static_assert(kMergePartials <= kMergedLeaves, "wave_total takes the partial sums of a bucket in one go");
int launch_dense_norms(QParams& p, const Shape& sh, const QuantizeArgs& a) {
    const uint64_t P = sh.N / kPartialTile;
    p.ws_tiles_per_worker = (uint32_t)(sh.nb * P);
    p.data_tiles = (sh.d + kPartialTile - 1) / kPartialTile;
    p.full_tiles = (uint32_t)(sh.d / kPartialTile);
    p.tail_tiles = (uint32_t)(p.data_tiles - p.full_tiles);
    p.xcd_group = xcd_group_log2(kPartialTile);
    p.merged = P <= kMergePartials;
    const dim3 grid((uint32_t)p.data_tiles, a.K);
    const uint32_t lds = stream_lds(p, 4, 16);
    if (p.center) hipLaunchKernelGGL(k_tile_partials_fast<true>, grid, dim3(256), lds, a.stream, p);
    else hipLaunchKernelGGL(k_tile_partials_fast<false>, grid, dim3(256), lds, a.stream, p);
    if (!p.merged) {
        uint32_t waves = 1;
        while (waves < 16 && (uint64_t)waves * 1024u < P) waves <<= 1;
        hipLaunchKernelGGL(k_finish_norms<QESGD_NORM_L2>, dim3((uint32_t)(sh.nb * a.K)), dim3(waves * kWaveSize), 0, a.stream, p, P, 1u);
    }
    return check_launch();
}

bool dense_wide(const Shape& sh, uint32_t norm_kind) {
    return sh.N > kMaxSinglePassBucket && norm_kind == QESGD_NORM_L2 && (sh.N == sh.B || sh.nb == 1);
}

int launch_quantize(const Shape& sh, const QuantizeArgs& a) {
    QParams p = quantize_params(sh, a);

    const uint64_t slots = sh.nb * sh.N;                 // slot space of one worker
    const bool two_pass = sh.N > kMaxSinglePassBucket;
    // Tiles that lie wholly inside the vector go to the fast kernel when the bucket is a
    // power of two (slot == coordinate), the scale is the L2 norm and the level width
    // divides a word (the other widths are served by the general kernels alone).
    const bool fast = !two_pass && a.norm_kind == QESGD_NORM_L2 && sh.N == sh.B && sh.log2N >= 5 &&
                      32u % sh.m == 0u;
    uint32_t ch = 2, nwaves = 4;                         // general kernels: 2 chunks per wave, 4..16 waves
    if (!two_pass && !fast) {
        if (sh.N == 8192) nwaves = 8;
        else if (sh.N == 16384) nwaves = 16;
        else if (sh.N == 32768) { ch = 4; nwaves = 16; }
    }
    const uint64_t tile = fast ? fast_tile(sh.m, sh.N, a.center != nullptr) : (uint64_t)nwaves * ch * kChunk;
    const uint64_t tiles = (slots + tile - 1) / tile;
    if (tiles * a.K >= (1ull << 31)) return QESGD_ERR_DIM;
    const dim3 block(nwaves * kWaveSize);
    p.log2_waves = nwaves == 16 ? 4 : nwaves == 8 ? 3 : 2;

    if (dense_wide(sh, a.norm_kind)) {
        // All workers at once in both passes: taking them in groups that fit the memory-side cache, with the
        // second pass walking backwards, cost a launch gap per group and pass and gained no bandwidth.
        const int rc = launch_dense_norms(p, sh, a);
        if (rc != QESGD_OK) return rc;
        launch_pre_fast(p, sh.m, dim3((uint32_t)p.data_tiles, a.K), a.stream);
        return check_launch();
    }
    if (two_pass) {
        // Buckets that are no power of two, and the max norm: all of slot space (over the
        // tiles that hold coordinates, where slot space equals coordinate space).
        const uint64_t P = sh.N / kPartialTile;          // tiles == nb * P
        uint32_t finish_waves = 1;
        while (finish_waves < 16 && (uint64_t)finish_waves * 1024u < P) finish_waves <<= 1;
        const bool dense = sh.N == sh.B || sh.nb == 1;
        p.ws_tiles_per_worker = (uint32_t)tiles;
        p.data_tiles = dense ? (sh.d + kPartialTile - 1) / kPartialTile : tiles;
        p.full_tiles = (uint32_t)p.data_tiles;
        p.xcd_group = xcd_group_log2(kPartialTile);
        const dim3 grid((uint32_t)p.data_tiles, a.K), finish_grid((uint32_t)(sh.nb * a.K)), finish_block(finish_waves * kWaveSize);
        if (a.norm_kind == QESGD_NORM_L2) {
            launch_partials<QESGD_NORM_L2>(p, grid, a.stream);
            hipLaunchKernelGGL(k_finish_norms<QESGD_NORM_L2>, finish_grid, finish_block, 0, a.stream, p, P, dense ? 1u : 0u);
        } else {
            launch_partials<QESGD_NORM_MAX>(p, grid, a.stream);
            hipLaunchKernelGGL(k_finish_norms<QESGD_NORM_MAX>, finish_grid, finish_block, 0, a.stream, p, P, dense ? 1u : 0u);
        }
        const int rc = check_launch();
        if (rc != QESGD_OK) return rc;
        launch_general<2, kPre>(p, sh.m, a.norm_kind, grid, block, a.stream);
        return check_launch();
    }

    if (fast) {
        // full_tiles may be 0 (a vector shorter than a tile): the launch is then one guarded tile per worker
        p.full_tiles = (uint32_t)(sh.d / tile);
        p.tail_tiles = (uint32_t)(tiles - p.full_tiles);
        p.xcd_group = xcd_group_log2(tile);
        launch_fast(p, sh.m, a.stream);
        return check_launch();
    }
    p.full_tiles = (uint32_t)tiles;
    p.xcd_group = xcd_group_log2(tile);
    p.codes_cached = general_codes_cached(sh, a.K, a.center != nullptr);
    const dim3 grid((uint32_t)tiles, a.K);
    if (ch == 4) launch_general<4, kBuckets>(p, sh.m, a.norm_kind, grid, block, a.stream);
    else if (sh.N >= 2 * kChunk) launch_general<2, kBuckets>(p, sh.m, a.norm_kind, grid, block, a.stream);
    else if (sh.N == sh.B || sh.nb == 1) launch_general<2, kNarrow>(p, sh.m, a.norm_kind, grid, block, a.stream);
    else launch_general<0, kNarrow>(p, sh.m, a.norm_kind, grid, block, a.stream);
    return check_launch();
}

}  // namespace qesgd
