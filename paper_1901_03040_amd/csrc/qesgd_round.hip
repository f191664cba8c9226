// A whole round in one launch, for one GPU that holds the K workers and the server: every
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
// where they do not (see round_fused_pays).  All vectors move in halves of a KiB per instruction, in runs
// of 64 K coordinates per XCD, with the non-temporal policy unless the round fits the memory-side cache and
// a wave owns one chunk; w and zsum are in flight while the last worker is rounded.  Before (32 bytes per
// lane, ordinary policy, tiles dealt round-robin, update loads after the last worker, z through LDS) / after:
//   d = 11 M, K = 8, s = 4, bucket 2048       118 ->  93 us = 6.6 TB/s
//   d = 12 M, K = 16, s = 256, bucket 8192    240 -> 199 us = 6.1 TB/s
//   d = 12 M, K = 2, s = 256, bucket 4096      70 ->  54 us
// The policy is chosen outside the loop over the workers: a branch inside it made every worker wait for the
// next one's coordinates (the three shapes above 102, 214 and 61 us; d = 2048, K = 8, s = 256, bucket 128 7.6 us,
// 6.9 without, 6.7 with the ordinary policy alone).
#include "qesgd_aggregate_device.h"
#include "qesgd_quantize_device.h"

namespace qesgd {
namespace {

struct RParams {
    QParams q;
    const float* w;
    float* zbar;
    float* u;
    float* zsum;
    float* z_acc;    // nullable (wide buckets only): z_acc += the mean
    float rcpK;      // exact 1/K when K is a power of two, else 0
    uint32_t K;
};

// Tile of a workgroup: chunks per wave and waves.  The running sum and the next worker's coordinates are
// held in registers next to the current ones, so fewer chunks fit than in the plain quantiser (two / one at
// d = 12 M, K = 8, bucket 4096, s = 256: 128 / 119 us; but 8192, s = 4: 128 / 141 us, where one would need
// sixteen waves).  Buckets of 16384 have 128 registers per lane and spill 44 to 80 bytes of them, 128 to 148 with a center: see round_fused_pays
// for where they take this kernel all the same.
template <int LOG2N>
struct RoundGeo {
    static constexpr int CH = LOG2N <= 12 ? 1 : 2;
    static constexpr int NW = LOG2N <= 10 ? 2 : (1 << LOG2N) / (CH * 512);
    static constexpr uint32_t TILE = (uint32_t)NW * CH * kChunk;
};
inline uint64_t round_tile(uint64_t N) { return N > 1024 ? N : 1024; }

template <int M, int LOG2N, bool CENTER, bool FULL, bool CACHED>
__device__ __forceinline__ void round_one_tile(const RParams& r, uint32_t t, float (&sm)[2][32]) {
    constexpr int CH = RoundGeo<LOG2N>::CH;
    constexpr uint32_t TILE = RoundGeo<LOG2N>::TILE;
    const QParams& p = r.q;
    FastCtx cx;
    cx.lane = threadIdx.x & 63u;
    cx.wave = threadIdx.x >> 6;
    cx.round = p.round;
    cx.key0 = p.key0;
    cx.key1 = p.key1;
    cx.smax = p.smax;
    cx.codes_cached = false;                              // nothing reads them here
    const uint32_t lane = cx.lane, first = cx.wave * (uint32_t)(CH * kChunk);
    const uint64_t o = (uint64_t)t * TILE + first;
    const uint32_t count = FULL ? TILE : (uint32_t)(p.d - (uint64_t)t * TILE), mine = FULL ? TILE : count_from(count, first);

    float acc[CH][8], v[CH][8];
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[c][e] = 0.0f;
    vec4 ca[CH], cb[CH], a[CH], b[CH], sa[CH], sb[CH];
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
        load_chunks_as<CH, FULL, CACHED>((last ? r.w : p.x + (uint64_t)(k + 1) * p.x_stride) + o, lane, mine, a, b);
        unsigned char* __restrict__ out = p.packed + (uint64_t)k * p.packed_stride;
        cx.norms = reinterpret_cast<float*>(out + p.norms_off);
        cx.signs = out + p.signs_off;
        cx.levels = out + p.levels_off;
        cx.worker = p.worker0 + k;
        process_tile<M, LOG2N, true, RoundGeo<LOG2N>, FULL>(cx, v, t, sm[k & 1u], acc, count);
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
        float z[8], u[8];                                 // v holds w
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            z[e] = (r.rcpK != 0.0f) ? acc[c][e] * r.rcpK : acc[c][e] / fk;
            u[e] = v[c][e] + z[e];
        }
        vec4 za, zb, ua, ub;
        lane_to_halves(z, za, zb);
        lane_to_halves(u, ua, ub);
        const uint64_t oc = o + (uint32_t)c * kChunk;
        const uint32_t left = FULL ? kChunk : count_from(mine, (uint32_t)c * kChunk);
        if (r.zbar) store_chunk<FULL>(r.zbar + oc, lane, left, za, zb);
        store_chunk<FULL>(r.u + oc, lane, left, ua, ub);
        if (r.zsum) store_chunk<FULL>(r.zsum + oc, lane, left, sa[c] + za, sb[c] + zb);
    }
}

template <int M, int LOG2N, bool CENTER>
__global__ void __launch_bounds__(RoundGeo<LOG2N>::NW * 64) k_round_fused(const RParams r) {
    __shared__ float sm[2][32];             // alternate per worker: one barrier per tile suffices
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x, r.q.xcd_group);
    // the policy is chosen once, outside the loop over the workers (see load_halves); with two chunks per wave
    // there is one form
    if (t >= r.q.full_tiles) round_one_tile<M, LOG2N, CENTER, false, true>(r, t, sm);   // the ragged last tile (at most one)
    else if (RoundGeo<LOG2N>::CH == 1 && r.q.x_cached) round_one_tile<M, LOG2N, CENTER, true, RoundGeo<LOG2N>::CH == 1>(r, t, sm);
    else round_one_tile<M, LOG2N, CENTER, true, false>(r, t, sm);
}

// The same behind the launches that found the scales of wide buckets: no wave needs another, so a wave owns
// 512 coordinates of every worker.  Lane k holds worker k's scale (from the norms plane, or finished from the
// partial sums by the workgroup's waves in turn) and hands it out as a scalar.  ZACC: z_acc += the mean.
// Bound by the stream of vectors; the codes are written but not read back.  Gradient round as four calls
// (partial sums, trees and codes per group of workers, mean, two updates) / as one call:
//   d = 853 K, K = 8, s = 256, one bucket     31.0 -> 21.3 us (partial sums, this; the chain of 8 workers)
//   d = 30 M, K = 4, s = 8, one bucket         378 -> 288 us
// (beyond about 1.2 GB, d = 25.6 M, K = 16 among them, the round takes two launches: see round_fused_pays)
// One wave per workgroup would finish every scale by itself; four share that work.
constexpr uint32_t kWideWaves = 4;

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
void launch_wide(const RParams& r, hipStream_t st) {
    const uint64_t blocks = (r.q.d + kWideWaves * kChunk - 1) / (kWideWaves * kChunk);
    const dim3 grid((uint32_t)blocks), block(kWideWaves * 64);
    if (r.z_acc) hipLaunchKernelGGL((k_round_wide<M, false, true>), grid, block, 0, st, r);
    else if (r.q.center) hipLaunchKernelGGL((k_round_wide<M, true, false>), grid, block, 0, st, r);
    else hipLaunchKernelGGL((k_round_wide<M, false, false>), grid, block, 0, st, r);
}

template <int M, int LOG2N>
void launch_one(const RParams& r, uint32_t blocks, hipStream_t st) {
    const dim3 grid(blocks), block(RoundGeo<LOG2N>::NW * 64);
    if (r.q.center) hipLaunchKernelGGL((k_round_fused<M, LOG2N, true>), grid, block, 0, st, r);
    else hipLaunchKernelGGL((k_round_fused<M, LOG2N, false>), grid, block, 0, st, r);
}

template <int M>
void launch_n(const RParams& r, uint32_t blocks, hipStream_t st) {
    switch (r.q.log2N) {
        case 5: launch_one<M, 5>(r, blocks, st); break;
        case 6: launch_one<M, 6>(r, blocks, st); break;
        case 7: launch_one<M, 7>(r, blocks, st); break;
        case 8: launch_one<M, 8>(r, blocks, st); break;
        case 9: launch_one<M, 9>(r, blocks, st); break;
        case 10: launch_one<M, 10>(r, blocks, st); break;
        case 11: launch_one<M, 11>(r, blocks, st); break;
        case 12: launch_one<M, 12>(r, blocks, st); break;
        case 13: launch_one<M, 13>(r, blocks, st); break;
        default: launch_one<M, 14>(r, blocks, st); break;
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

}  // namespace

bool round_fused_covers(const Shape& sh, uint32_t norm_kind) {
    if (dense_wide(sh, norm_kind)) return true;
    return norm_kind == QESGD_NORM_L2 && sh.N == sh.B && sh.log2N >= 5 && sh.N <= 16384 &&
           32u % sh.m == 0u;
}

int launch_round_fused(const Shape& sh, const QuantizeArgs& a, const AggregateArgs& g) {
    RParams r{};
    QParams& p = r.q;
    p = quantize_params(sh, a);
    r.w = g.w_snap;
    r.zbar = g.zbar_out;
    r.u = g.u_out;
    r.zsum = g.zsum;
    r.z_acc = g.z_acc;
    r.K = a.K;
    r.rcpK = ((a.K & (a.K - 1)) == 0) ? 1.0f / (float)a.K : 0.0f;
    if (sh.N > kMaxSinglePassBucket) {
        const int rc = launch_dense_norms(p, sh, a);
        if (rc != QESGD_OK) return rc;
        p.xcd_group = xcd_group_log2(kWideWaves * kChunk);
        switch (sh.m) {
            case 1: launch_wide<1>(r, a.stream); break;
            case 2: launch_wide<2>(r, a.stream); break;
            case 3: launch_wide<3>(r, a.stream); break;
            case 4: launch_wide<4>(r, a.stream); break;
            case 5: launch_wide<5>(r, a.stream); break;
            case 6: launch_wide<6>(r, a.stream); break;
            case 7: launch_wide<7>(r, a.stream); break;
            case 8: launch_wide<8>(r, a.stream); break;
            default: launch_wide<16>(r, a.stream); break;
        }
        return check_launch();
    }
    const uint64_t tile = round_tile(sh.N);
    const uint64_t tiles = (sh.nb * sh.N + tile - 1) / tile;
    if (tiles >= (1ull << 31)) return QESGD_ERR_DIM;
    p.full_tiles = (uint32_t)(sh.d / tile);
    p.tail_tiles = (uint32_t)(tiles - p.full_tiles);
    p.xcd_group = xcd_group_log2(tile);
    switch (sh.m) {
        case 1: launch_n<1>(r, (uint32_t)tiles, a.stream); break;
        case 2: launch_n<2>(r, (uint32_t)tiles, a.stream); break;
        case 4: launch_n<4>(r, (uint32_t)tiles, a.stream); break;
        case 8: launch_n<8>(r, (uint32_t)tiles, a.stream); break;
        default: launch_n<16>(r, (uint32_t)tiles, a.stream); break;
    }
    return check_launch();
}

}  // namespace qesgd
