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
// where they do not (see round_fused_pays).  All vectors move in halves of a KiB per instruction with
// the non-temporal policy, in runs of 64 K coordinates per XCD; w and zsum are in flight while the last
// worker is rounded.  Before (32 bytes per lane, ordinary policy, tiles dealt round-robin, update loads
// after the last worker, z through LDS) / after:
//   d = 11 M, K = 8, s = 4, bucket 2048       118 -> 102 us = 6.0 TB/s
//   d = 12 M, K = 16, s = 256, bucket 8192    245 -> 220 us = 5.7 TB/s
//   d = 12 M, K = 2, s = 256, bucket 4096      73 ->  60 us
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
    float rcpK;      // exact 1/K when K is a power of two, else 0
    uint32_t K;
};

// Tile of a workgroup: chunks per wave and waves.  The running sum and the next worker's coordinates are
// held in registers next to the current ones, so fewer chunks fit than in the plain quantiser (two
// chunks at bucket 2048, s = 4: 115 against 111 us at d = 11 M, K = 8).
template <int LOG2N>
struct RoundGeo {
    static constexpr int CH = LOG2N <= 11 ? 1 : 2;
    static constexpr int NW = (LOG2N <= 10) ? 2 : ((LOG2N <= 12) ? 4 : (LOG2N == 13 ? 8 : 16));
    static constexpr uint32_t TILE = (uint32_t)NW * CH * kChunk;
};
inline uint64_t round_tile(uint64_t N) { return N > 2048 ? (N > 4096 ? N : 4096) : (N > 1024 ? N : 1024); }

template <int M, int LOG2N, bool CENTER>
__global__ void __launch_bounds__(RoundGeo<LOG2N>::NW * 64) k_round_fused(const RParams r) {
    constexpr int CH = RoundGeo<LOG2N>::CH;
    constexpr uint32_t TILE = RoundGeo<LOG2N>::TILE;
    __shared__ float sm[2][32];             // alternate per worker: one barrier per tile suffices
    const QParams& p = r.q;
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x, p.xcd_group);
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;

    float acc[CH][8];
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[c][e] = 0.0f;

    if (t < p.full_tiles) {
        const uint64_t o = (uint64_t)t * TILE + wave * (uint32_t)(CH * kChunk) + half_offset(lane);
        // one branch per worker for the policy is free with one chunk per wave (99 against 103 us at d = 11 M,
        // K = 8, bucket 2048) and costs 8% with two
        const bool cached = CH == 1 && p.x_cached;
        vec4 ca[CH], cb[CH], a[CH], b[CH], na[CH], nb[CH], sa[CH], sb[CH];
        if (CENTER) load_halves<CH>(p.center + o, false, ca, cb);
        load_halves<CH>(p.x + o, cached, a, b);
        for (uint32_t k = 0; k < r.K; ++k) {
            // in flight while worker k is rounded: the next worker's coordinates, after the last the update's
            const bool last = k + 1 == r.K;
            load_halves<CH>((last ? r.w : p.x + (uint64_t)(k + 1) * p.x_stride) + o, cached, na, nb);
            if (last && r.zsum) load_halves<CH>(r.zsum + o, cached, sa, sb);
            float v[CH][8];
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                if (CENTER) halves_to_lane(a[c] - ca[c], b[c] - cb[c], v[c]);
                else halves_to_lane(a[c], b[c], v[c]);
            }
            unsigned char* __restrict__ out = p.packed + (uint64_t)k * p.packed_stride;
            FastCtx cx;
            cx.norms = reinterpret_cast<float*>(out + p.norms_off);
            cx.signs = out + p.signs_off;
            cx.levels = out + p.levels_off;
            cx.lane = lane;
            cx.wave = wave;
            cx.worker = p.worker0 + k;
            cx.round = p.round;
            cx.key0 = p.key0;
            cx.key1 = p.key1;
            cx.smax = p.smax;
            cx.codes_cached = false;                     // nothing reads them here
            process_tile<M, LOG2N, true, RoundGeo<LOG2N>>(cx, v, t, sm[k & 1u], acc);
#pragma unroll
            for (int c = 0; c < CH; ++c) { a[c] = na[c]; b[c] = nb[c]; }
        }
        const float fk = (float)r.K;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            float z[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) z[e] = (r.rcpK != 0.0f) ? acc[c][e] * r.rcpK : acc[c][e] / fk;
            vec4 za, zb;
            lane_to_halves(z, za, zb);
            const uint64_t ia = o + (uint32_t)c * kChunk, ib = ia + kChunk / 2;
            if (r.zbar) {
                store_stream(r.zbar + ia, za);
                store_stream(r.zbar + ib, zb);
            }
            store_stream(r.u + ia, a[c] + za);
            store_stream(r.u + ib, b[c] + zb);
            if (r.zsum) {
                store_stream(r.zsum + ia, sa[c] + za);
                store_stream(r.zsum + ib, sb[c] + zb);
            }
        }
        return;
    }

    // the ragged last tile
    LaneSpan span[CH];
    float v[CH][8];
    guarded_spans<CH>(p, t, span);
    for (uint32_t k = 0; k < r.K; ++k) {
        guarded_load<CH>(p, k, span, v);
        guarded_codes<M, CH, QESGD_NORM_L2, false, true>(p, k, span, v, sm[k & 1u], acc);
    }
    const float fk = (float)r.K;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        // the ragged tile, lane by lane (power-of-two buckets: slot == coordinate)
        const uint64_t i = (uint64_t)t * TILE + (wave * (uint32_t)CH + (uint32_t)c) * kChunk + lane * kLaneElems;
        if (i >= p.d) continue;
        const uint64_t rem = p.d - i;
        const uint32_t nvalid = rem < 8 ? (uint32_t)rem : 8u;
        float z[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = (r.rcpK != 0.0f) ? acc[c][e] * r.rcpK : acc[c][e] / fk;
        if (r.zbar) store8(r.zbar, i, nvalid, z);
        float w8[8], u8[8];
        load8(r.w, i, nvalid, w8);
#pragma unroll
        for (int e = 0; e < 8; ++e) u8[e] = w8[e] + z[e];
        store8(r.u, i, nvalid, u8);
        if (r.zsum) {
            float s8[8];
            load8(r.zsum, i, nvalid, s8);
#pragma unroll
            for (int e = 0; e < 8; ++e) s8[e] = s8[e] + z[e];
            store8(r.zsum, i, nvalid, s8);
        }
    }
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

}  // namespace

bool round_fused_covers(const Shape& sh, uint32_t norm_kind) {
    return norm_kind == QESGD_NORM_L2 && sh.N == sh.B && sh.log2N >= 5 && sh.N <= 16384 &&
           32u % sh.m == 0u;
}

int launch_round_fused(const Shape& sh, const QuantizeArgs& a, const AggregateArgs& g) {
    RParams r{};
    QParams& p = r.q;
    p.x = a.x;
    p.center = a.center;
    p.packed = a.packed;
    p.x_stride = a.x_stride;
    p.packed_stride = a.packed_stride;
    p.d = sh.d;
    p.B = sh.B;
    p.nb = sh.nb;
    p.norms_off = sh.lay.norms_off;
    p.signs_off = sh.lay.signs_off;
    p.levels_off = sh.lay.levels_off;
    p.log2N = sh.log2N;
    p.key0 = (uint32_t)a.seed;
    p.key1 = (uint32_t)(a.seed >> 32);
    p.round = a.round;
    p.worker0 = a.worker0;
    p.smax = (float)(sh.s - 1);
    p.group_workers = a.K;
    p.x_cached = input_cached(sh, a.K);
    const uint64_t tile = round_tile(sh.N);
    const uint64_t tiles = (sh.nb * sh.N + tile - 1) / tile;
    if (tiles >= (1ull << 31)) return QESGD_ERR_DIM;
    p.full_tiles = (uint32_t)(sh.d / tile);
    p.tail_tiles = (uint32_t)(tiles - p.full_tiles);
    p.xcd_group = xcd_group_log2(tile);
    r.w = g.w_snap;
    r.zbar = g.zbar_out;
    r.u = g.u_out;
    r.zsum = g.zsum;
    r.K = a.K;
    r.rcpK = ((a.K & (a.K - 1)) == 0) ? 1.0f / (float)a.K : 0.0f;
    switch (sh.m) {
        case 1: launch_n<1>(r, (uint32_t)tiles, a.stream); break;
        case 2: launch_n<2>(r, (uint32_t)tiles, a.stream); break;
        case 4: launch_n<4>(r, (uint32_t)tiles, a.stream); break;
        case 8: launch_n<8>(r, (uint32_t)tiles, a.stream); break;
        default: launch_n<16>(r, (uint32_t)tiles, a.stream); break;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_last_hip_error((int)e);
        return QESGD_ERR_HIP;
    }
    return QESGD_OK;
}

}  // namespace qesgd
