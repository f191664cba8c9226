// Kernels of a whole round in one launch (not installed), for one GPU that holds the K workers and the server: every
// worker's quantise + pack (Sec. 2.1, Eq. (2); Sec. 3) and the server's sum over workers and
// update (Alg. 3, server task; Alg. 2: u = w_t + z) with the results of the two-call form, bit
// for bit, including the packed blocks.
//
// No grid-wide wait is needed: buckets are independent on the worker side and coordinates on the
// server side, so a workgroup that owns one tile of every worker has all it needs for that tile of
// z.  It takes the workers one after the other (the next worker's loads in flight while the
// current one is rounded), keeps the running sum of the dequantised codes in registers, and writes
// z, u and the running sum of z at the end.  The packed codes are written but never read back.
// What this saves is one dependent launch per round and K*P bytes of reads.
//
// Bound by the stream of vectors where the tiles fill the chip, by the chain of K workers per tile
// where they do not (see round_chunks).  All vectors move in halves of a KiB per instruction, in runs
// of 64 K coordinates per XCD, with the non-temporal policy unless the round fits the memory-side cache and
// a wave owns one chunk; w and zsum are in flight while the last worker is rounded.  Before (32 bytes per
// lane, ordinary policy, tiles dealt round-robin, update loads after the last worker, z through LDS) / after:
//   d = 11 M, K = 8, s = 4, bucket 2048       118 ->  93 us = 6.6 TB/s
//   d = 12 M, K = 16, s = 256, bucket 8192    240 -> 199 us = 6.1 TB/s
//   d = 12 M, K = 2, s = 256, bucket 4096      70 ->  54 us
// The policy is chosen outside the loop over the workers: a branch inside it made every worker wait for the
// next one's coordinates (the three shapes above 102, 214 and 61 us; d = 2048, K = 8, s = 256, bucket 128 7.6 us,
// 6.9 without, 6.7 with the ordinary policy alone).
// Level widths of 3, 5, 6 and 7 bits and the running mean of a gradient round (ZACC), two launches / this:
//   d = 25.6 M, K = 16, s = 128, bucket 2048        540 -> 472 us
//   d = 11 M, K = 8, s = 32, bucket 1024            119 -> 101 us
//   gradient, d = 11 M, K = 8, s = 4, bucket 1024   118 -> 111 us
//   gradient, d = 2000, K = 4, s = 256, bucket 128  9.0 -> 6.4 us
#pragma once

#include "qesgd_aggregate_device.h"
#include "qesgd_round.h"

namespace qesgd {

namespace {

// Tile of a workgroup: chunks per wave and waves.  The running sum and the next worker's coordinates are
// held in registers next to the current ones, so fewer chunks fit than in the plain quantiser: one up to 4096, where two
// pay only beyond the caches (see round_chunks).  Registers, level widths that divide 32 / 3, 5, 6, 7: one chunk 75 to 94 /
// 86 to 107, two 139 to 163.  Buckets of 8192 and 16384 have two, one would need sixteen waves and more (8192, d = 12 M,
// K = 8, s = 4: 128 / 141 us).  Those of 8192 take 137 to 158 / 151 to 178, those of 16384 have 128 per lane and spill
// 44 to 80 / 124 bytes and more of them, with a center or z_acc 116 to 200.
template <int LOG2N, int CHUNKS>
struct RoundGeo {
    static constexpr int CH = CHUNKS;
    static constexpr int NW = (1 << LOG2N) <= 2 * CH * 512 ? 2 : (1 << LOG2N) / (CH * 512);
    static constexpr uint32_t TILE = (uint32_t)NW * CH * kChunk;
};

template <int M, int LOG2N, class G, bool CENTER, bool ZACC, bool FULL, bool CACHED>
__device__ __forceinline__ void round_one_tile(const RParams& r, uint32_t t, float (&sm)[2][32], unsigned char* string) {
    constexpr int CH = G::CH;
    constexpr uint32_t TILE = G::TILE;
    const QParams& p = r.q;
    FastCtx cx;
    cx.lane = threadIdx.x & 63u;
    cx.wave = threadIdx.x >> 6;
    cx.round = p.round;
    cx.key0 = p.key0;
    cx.key1 = p.key1;
    cx.smax = p.smax;
    cx.codes_cached = false;                              // nothing reads them here
    cx.string = string;
    const uint32_t lane = cx.lane, first = cx.wave * (uint32_t)(CH * kChunk);
    const uint64_t o = (uint64_t)t * TILE + first;
    const uint32_t count = FULL ? TILE : (uint32_t)(p.d - (uint64_t)t * TILE), mine = FULL ? TILE : count_from(count, first);

    float acc[CH][8], v[CH][8];
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[c][e] = 0.0f;
    vec4 ca[CH], cb[CH], a[CH], b[CH], sa[CH], sb[CH], ta[CH], tb[CH];
    load_chunks_as<CH, FULL, CACHED>(p.x + o, lane, mine, a, b);
    if (CENTER) load_chunks_as<CH, FULL, false>(p.center + o, lane, mine, ca, cb);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (CENTER) halves_to_lane(a[c] - ca[c], b[c] - cb[c], v[c]);
        else halves_to_lane(a[c], b[c], v[c]);
    }
    for (uint32_t k = 0; k < r.K; ++k) {
        // in flight while worker k is rounded: the next worker's coordinates, after the last the update's
        const bool last = k + 1 == r.K;
        if (last && r.zsum) load_chunks_as<CH, FULL, CACHED>(r.zsum + o, lane, mine, sa, sb);
        if (last && ZACC) load_chunks_as<CH, FULL, CACHED>(r.z_acc + o, lane, mine, ta, tb);
        load_chunks_as<CH, FULL, CACHED>((last ? r.w : p.x + (uint64_t)(k + 1) * p.x_stride) + o, lane, mine, a, b);
        unsigned char* __restrict__ out = p.packed + (uint64_t)k * p.packed_stride;
        cx.norms = reinterpret_cast<float*>(out + p.norms_off);
        cx.signs = out + p.signs_off;
        cx.levels = out + p.levels_off;
        cx.worker = p.worker0 + k;
        process_tile<M, LOG2N, true, G, FULL>(cx, v, t, sm[k & 1u], acc, count);
        // the exchange stands at the end of the worker's work: it is what waits for the loads
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (CENTER && !last) {
                a[c] -= ca[c];
                b[c] -= cb[c];
            }
            halves_to_lane(a[c], b[c], v[c]);
        }
    }
    const float fk = (float)r.K;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        float z[8];                                       // v holds w
        vec4 za, zb, ua, ub;
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = (r.rcpK != 0.0f) ? acc[c][e] * r.rcpK : acc[c][e] / fk;
        if (!ZACC) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[c][e] = v[c][e] + z[e];
        }
        lane_to_halves(z, za, zb);
        lane_to_halves(v[c], ua, ub);
        const uint64_t oc = o + (uint32_t)c * kChunk;
        const uint32_t left = FULL ? kChunk : count_from(mine, (uint32_t)c * kChunk);
        if (r.zbar) store_chunk<FULL>(r.zbar + oc, lane, left, za, zb);
        if (ZACC) {
            za = ta[c] + za;
            zb = tb[c] + zb;
            store_chunk<FULL>(r.z_acc + oc, lane, left, za, zb);
            ua = ua + za;
            ub = ub + zb;
        }
        store_chunk<FULL>(r.u + oc, lane, left, ua, ub);
        if (r.zsum) store_chunk<FULL>(r.zsum + oc, lane, left, sa[c] + za, sb[c] + zb);
    }
}

template <int M, int LOG2N, int CH, bool CENTER, bool ZACC>
__global__ void __launch_bounds__((RoundGeo<LOG2N, CH>::NW * 64)) k_round_fused(const RParams r) {
    typedef RoundGeo<LOG2N, CH> G;
    __shared__ float sm[2][32];             // alternate per worker: one barrier per tile suffices
    __shared__ __align__(16) unsigned char strings[32 % M == 0 ? 16 : G::NW * kStringBytes<M>];
    unsigned char* string = strings + (threadIdx.x >> 6) * kStringBytes<M>;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x, r.q.xcd_group);
    // the policy is chosen once, outside the loop over the workers (see load_halves); with two chunks per wave
    // there is one form
    if (t >= r.q.full_tiles) round_one_tile<M, LOG2N, G, CENTER, ZACC, false, true>(r, t, sm, string);   // the ragged last tile (at most one)
    else if (CH == 1 && r.q.x_cached) round_one_tile<M, LOG2N, G, CENTER, ZACC, true, CH == 1>(r, t, sm, string);
    else round_one_tile<M, LOG2N, G, CENTER, ZACC, true, false>(r, t, sm, string);
}

// The same behind the launches that found the scales of wide buckets: no wave needs another, so a wave owns
// 512 coordinates of every worker.  Lane k holds worker k's scale (from the norms plane, or finished from the
// partial sums by the workgroup's waves in turn) and hands it out as a scalar.  ZACC: z_acc += the mean.
// Bound by the stream of vectors; the codes are written but not read back.  Gradient round as four calls
// (partial sums, trees and codes per group of workers, mean, two updates) / as one call:
//   d = 853 K, K = 8, s = 256, one bucket     31.0 -> 21.3 us (partial sums, this; the chain of 8 workers)
//   d = 30 M, K = 4, s = 8, one bucket         378 -> 288 us
// (beyond about 1.2 GB, d = 25.6 M, K = 16 among them, the round takes two launches: see round_chunks)
// One wave per workgroup would finish every scale by itself; four (kWideWaves) share that work.

// string: kStringBytes<M> of LDS that are the wave's.  norm: lane k holds worker k's (lanes from K on: 1).  ca, cb, a, b: the center's and the first worker's.
template <int M, bool CENTER, bool ZACC, bool FULL>
__device__ __forceinline__ void wide_chunk(const RParams& r, unsigned char* string, uint64_t c0, uint32_t lane, float norm, const vec4 (&ca)[1],
                                           const vec4 (&cb)[1], vec4 (&a)[1], vec4 (&b)[1]) {
    const QParams& p = r.q;
    const uint32_t count = FULL ? kChunk : (uint32_t)(p.d - c0);
    const bool cached = p.x_cached;
    const float my_step = norm / p.smax, my_mul = scale_of_norm<M>(norm).mul;
    const uint64_t direct = __builtin_amdgcn_ballot_w64(norm >= 0x1p-60f && norm <= 0x1p60f);
    const uint64_t g0 = c0 / kLaneElems;
    vec4 na[1], nb[1], sa[1], sb[1], ta[1], tb[1];
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
    for (uint32_t k = 0; k < r.K; ++k) {
        const bool last = k + 1 == r.K;
        // (a choice in the loop, unlike in round_one_tile: two copies of the loop were slower here, 19.6 against
        // 18.6 us at d = 853 K, K = 8, s = 256)
        load_chunks<1, FULL>((last ? r.w : p.x + (uint64_t)(k + 1) * p.x_stride) + c0, lane, count, cached, na, nb);
        if (last && r.zsum) load_chunks<1, FULL>(r.zsum + c0, lane, count, cached, sa, sb);
        if (last && ZACC) load_chunks<1, FULL>(r.z_acc + c0, lane, count, cached, ta, tb);
        float v[8];
        if (CENTER) halves_to_lane(a[0] - ca[0], b[0] - cb[0], v);
        else halves_to_lane(a[0], b[0], v);
        Scale sc;
        sc.norm = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(norm), k));
        sc.mul = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_mul), k));
        sc.direct = (direct >> k) & 1u;
        const float step = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_step), k));
        uint32_t rnd[4], sign_byte, bits[4];
        philox4x32_10((uint32_t)g0 + lane, (uint32_t)(g0 >> 32), p.worker0 + k, p.round, p.key0, p.key1, rnd);
        round_and_pack<M>(v, rnd, sc, sign_byte, bits);
        unsigned char* __restrict__ out = p.packed + (uint64_t)k * p.packed_stride;
        if (FULL) {
            store_whole<M>(string, out + p.signs_off, out + p.levels_off, c0, lane, false, sign_byte, bits);
        } else {
            const uint32_t before = lane * kLaneElems;
            const uint32_t nvalid = before < count ? (count - before < 8u ? count - before : 8u) : 0u;
            store_codes<M>(reinterpret_cast<uint32_t*>(out + p.signs_off), reinterpret_cast<uint32_t*>(out + p.levels_off),
                           c0 + before, nvalid, lane, sign_byte, bits);
        }
        accumulate8<M>(acc, sign_byte, bits, step);
        a[0] = na[0];
        b[0] = nb[0];
    }
    const float fk = (float)r.K;
    float z[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = (r.rcpK != 0.0f) ? acc[e] * r.rcpK : acc[e] / fk;
    vec4 za, zb;
    lane_to_halves(z, za, zb);
    if (r.zbar) store_chunk<FULL>(r.zbar + c0, lane, count, za, zb);
    if (ZACC) {
        za = ta[0] + za;
        zb = tb[0] + zb;
        store_chunk<FULL>(r.z_acc + c0, lane, count, za, zb);
    }
    store_chunk<FULL>(r.u + c0, lane, count, a[0] + za, b[0] + zb);
    if (r.zsum) store_chunk<FULL>(r.zsum + c0, lane, count, sa[0] + za, sb[0] + zb);
}

template <int M, bool CENTER, bool ZACC>
__global__ void __launch_bounds__(kWideWaves * 64) k_round_wide(const RParams r) {
    __shared__ float total[64];
    __shared__ __align__(16) unsigned char strings[kWideWaves][kStringBytes<M> + 16];
    const QParams& p = r.q;
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x, p.xcd_group) * kWideWaves + wave;
    const uint64_t c0 = (uint64_t)t * kChunk;             // first coordinate of the wave
    const bool full = c0 + kChunk <= p.d;
    vec4 ca[1], cb[1], a[1], b1[1];
    if (full) {
        if (CENTER) load_chunks<1, true>(p.center + c0, lane, kChunk, false, ca, cb);
        load_chunks<1, true>(p.x + c0, lane, kChunk, p.x_cached, a, b1);
    }

    float norm = 1.0f;
    if (p.merged) {                                       // the workgroup's waves lie in one bucket (a multiple of 32768, or the only one)
        const uint64_t first = (uint64_t)(t - wave) * kChunk;
        const uint32_t P = 1u << (p.log2N - 12u);
        const uint64_t b = first >> p.log2N, left = p.data_tiles - b * P;
        for (uint32_t k = wave; k < r.K; k += kWideWaves) {
            const float sum = wave_total<QESGD_NORM_L2>(p.workspace + (uint64_t)k * p.ws_tiles_per_worker + b * P, P,
                                                        left < P ? (uint32_t)left : P, lane);
            if (lane == 0) total[k] = sum;
        }
        __syncthreads();
        if (lane < r.K) {
            norm = sqrtf(total[lane]);
            if (wave == 0 && first == b << p.log2N)
                reinterpret_cast<float*>(p.packed + (uint64_t)lane * p.packed_stride + p.norms_off)[b] = norm;
        }
    } else if (lane < r.K && c0 < p.d) {
        norm = reinterpret_cast<const float*>(p.packed + (uint64_t)lane * p.packed_stride + p.norms_off)[c0 >> p.log2N];
    }
    if (full) {
        wide_chunk<M, CENTER, ZACC, true>(r, strings[wave], c0, lane, norm, ca, cb, a, b1);
    } else if (c0 < p.d) {                                // ragged last wave
        const uint32_t count = (uint32_t)(p.d - c0);
        if (CENTER) load_chunks<1, false>(p.center + c0, lane, count, true, ca, cb);
        load_chunks<1, false>(p.x + c0, lane, count, true, a, b1);
        wide_chunk<M, CENTER, ZACC, false>(r, strings[wave], c0, lane, norm, ca, cb, a, b1);
    }
}

template <int M>
void launch_wide(const RParams& r, uint32_t blocks, hipStream_t st) {
    const dim3 grid(blocks), block(kWideWaves * 64);
    if (r.z_acc) hipLaunchKernelGGL((k_round_wide<M, false, true>), grid, block, 0, st, r);
    else if (r.q.center) hipLaunchKernelGGL((k_round_wide<M, true, false>), grid, block, 0, st, r);
    else hipLaunchKernelGGL((k_round_wide<M, false, false>), grid, block, 0, st, r);
}

template <int M, int LOG2N, int CH>
void launch_one(const RParams& r, uint32_t blocks, hipStream_t st) {
    const dim3 grid(blocks), block(RoundGeo<LOG2N, CH>::NW * 64);
    if (r.z_acc) hipLaunchKernelGGL((k_round_fused<M, LOG2N, CH, false, true>), grid, block, 0, st, r);
    else if (r.q.center) hipLaunchKernelGGL((k_round_fused<M, LOG2N, CH, true, false>), grid, block, 0, st, r);
    else hipLaunchKernelGGL((k_round_fused<M, LOG2N, CH, false, false>), grid, block, 0, st, r);
}
template <int M, int LOG2N>
void launch_ch(const RParams& r, uint32_t chunks, uint32_t blocks, hipStream_t st) {
    if constexpr (LOG2N > 12) {
        launch_one<M, LOG2N, 2>(r, blocks, st);
    } else {
        if constexpr (M >= 4 && 32 % M == 0) {
            if (chunks == 2) {
                launch_one<M, LOG2N, 2>(r, blocks, st);
                return;
            }
        }
        launch_one<M, LOG2N, 1>(r, blocks, st);
    }
}

}  // namespace

template <int M>
void launch_round(const RParams& r, uint32_t chunks, uint32_t blocks, hipStream_t st) {
    if (chunks == 0) {
        launch_wide<M>(r, blocks, st);
        return;
    }
    switch (r.q.log2N) {
        case 5: launch_ch<M, 5>(r, chunks, blocks, st); break;
        case 6: launch_ch<M, 6>(r, chunks, blocks, st); break;
        case 7: launch_ch<M, 7>(r, chunks, blocks, st); break;
        case 8: launch_ch<M, 8>(r, chunks, blocks, st); break;
        case 9: launch_ch<M, 9>(r, chunks, blocks, st); break;
        case 10: launch_ch<M, 10>(r, chunks, blocks, st); break;
        case 11: launch_ch<M, 11>(r, chunks, blocks, st); break;
        case 12: launch_ch<M, 12>(r, chunks, blocks, st); break;
        case 13: launch_ch<M, 13>(r, chunks, blocks, st); break;
        default: launch_ch<M, 14>(r, chunks, blocks, st); break;
    }
}

}  // namespace qesgd
