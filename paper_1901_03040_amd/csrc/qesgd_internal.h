// Internal declarations shared by the translation units of libqesgd (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qesgd.h"

namespace qesgd {

// Coordinates handled by one lane per chunk, lanes per wavefront, and the
// resulting wave chunk: 64 lanes x 8 consecutive coordinates.
constexpr uint32_t kLaneElems = 8;
constexpr uint32_t kWaveSize = 64;
constexpr uint32_t kChunk = kLaneElems * kWaveSize;   // 512

// Largest zero-padded bucket whose scale is found in the same pass that
// quantises it (16 waves x 4 chunks x 512 coordinates held in registers).
constexpr uint64_t kMaxSinglePassBucket = 32768;
// Tile of the partial-sum pass used for larger buckets.
constexpr uint64_t kPartialTile = 4096;
// Cache policy of the streams.  The non-temporal one is right for what comes from HBM; what fits the
// 256 MB memory-side cache from one round to the next, or from the workers' call to the server's, is
// better read and written with the ordinary one.  Measured over d = 0.3 .. 12 M, K = 2 .. 16, with two
// rounds' buffers in turn (whole two-call round, non-temporal / ordinary):
//   input vectors                  d = 2 M, K = 8: 23.9 / 22.1 us;  d = 8 M, K = 8: 80.8 / 83.9 us
//   level planes                   d = 5 M, K = 16, s = 256: 103 / 94 us;  12 M (216 MB): 234 / 237 us
//   w and zsum of the update       d = 5 M, K = 4: 34.9 / 31.9 us;  12 M, K = 16, s = 256: 234 / 239 us
// (the outputs z, u and zsum are best non-temporal at every size).
constexpr uint64_t kCachedInputBytes = 96ull << 20;     // of the K input vectors ...
constexpr uint64_t kCachedRoundBytes = 192ull << 20;    // ... and of all that a round touches
constexpr uint64_t kCachedCodeBytes = 160ull << 20;     // of the K packed blocks, which the server reads next
constexpr uint64_t kCachedUpdateBytes = 256ull << 20;   // of the packed blocks and the five vectors of the update
// The update alone (qesgd_apply_update), of its three or four vectors; non-temporal / ordinary, loads and stores, two
// sets of vectors in turn: with zsum d = 5 M 16.5 / 14.8 us, 8 M 25.4 / 23.3, 10 M 31.5 / 31.3, 16 M 50.0 / 57.6;
// without d = 8 M 15.6 / 14.7, 12 M 22.9 / 23.3, 25 M 46.6 / 52.2.
constexpr uint64_t kCachedApplyBytes = 128ull << 20;
// Floats of the per-GPU static scratch behind qesgd_quantize_pack_batched_noalloc (4 MiB): one
// partial sum per 4096 padded coordinates, i.e. K * n_buckets * padded_bucket <= 2^32.
constexpr size_t kStaticScratchFloats = QESGD_NOALLOC_SCRATCH_BYTES / sizeof(float);

struct Shape {
    uint64_t d;
    uint32_t s;
    uint32_t m;          // level bits
    uint64_t B;          // effective bucket = min(bucket, d)
    uint64_t nb;         // buckets
    uint64_t N;          // B zero-padded to a power of two, at least 8
    uint32_t log2N;
    qesgd_layout lay;
};

// Validates (d, s, bucket) and fills the shape; returns QESGD_OK or an error.
int make_shape(uint64_t d, uint32_t s, uint64_t bucket, Shape* out);

// What the K workers' vectors, their packed blocks and the update's five vectors take.
inline uint64_t update_bytes(const Shape& sh, uint32_t K) { return K * sh.lay.payload_bytes + 20u * sh.d; }
inline bool input_cached(const Shape& sh, uint32_t K) {
    const uint64_t in = 4u * (uint64_t)K * sh.d;
    return in <= kCachedInputBytes && in + update_bytes(sh, K) <= kCachedRoundBytes;
}

struct QuantizeArgs {
    const float* x;
    uint64_t x_stride;       // floats between workers
    const float* center;     // nullable
    uint32_t norm_kind;
    uint64_t seed;
    uint32_t round;
    uint32_t worker0;        // worker id of slab row 0
    uint32_t K;              // rows
    unsigned char* packed;
    uint64_t packed_stride;  // bytes between workers
    float* workspace;        // two-pass path only
    hipStream_t stream;
};

struct AggregateArgs {
    const unsigned char* packed;
    uint64_t packed_stride;
    uint32_t K;
    const float* w_snap;     // nullable: no update
    float* zbar_out;         // nullable
    float* u_out;            // nullable iff w_snap is
    float* zsum;             // nullable
    float* z_acc;            // nullable: z_acc += the mean, and z_acc takes the mean's place in u and zsum
    hipStream_t stream;
};

int launch_quantize(const Shape& sh, const QuantizeArgs& a);
// Device address of the current GPU's static scratch (kStaticScratchFloats floats).
int static_scratch(float** out);
int launch_aggregate(const Shape& sh, const AggregateArgs& a);
// Wide buckets whose slot space equals coordinate space (a power of two, or a single bucket), L2 scale.
bool dense_wide(const Shape& sh, uint32_t norm_kind);
// One launch for a whole round (quantise K workers, sum, update) where the shape allows it:
// power-of-two bucket of 32..16384 coordinates, L2 scale, level width dividing 32; or, behind the launches
// that find the scales, a dense wide bucket with the L2 scale.
bool round_fused_covers(const Shape& sh, uint32_t norm_kind);
// One launch or two.  One launch takes the workers of a tile one after the other, about 1 us each (2.4 us
// with buckets of 4096 and more, whose waves meet at a barrier per worker), which only a chip full of
// tiles hides; two launches spread tiles and workers over the chip at once.  Measured, one / two, whole round:
//   from 1.5 M coordinates on       1.7 M, K = 16, bucket 512: 32.1 / 34.8 us; 1.7 M, K = 4, bucket 8192: 14.1 / 15.9;
//                                   12 M, K = 16, bucket 8192: 183 / 187; 12 M, K = 8, bucket 16384: 126 / 129
//     (with 8192 and 16384 two would be better up to about 10 M: 2.4 M, K = 8, bucket 8192 34.8 / 26.1; 5 M, K = 8,
//     54 / 48; 1.7 M, K = 8, bucket 16384 31.5 / 22.4; not so with K = 1, 2: 2.4 M, K = 2, bucket 16384 14.2 / 17.4)
//   below, up to 8 workers          1 M, K = 8, bucket 512: 11.0 / 14.6; 0.1 M, K = 8, bucket 64: 7.6 / 7.2
//     up to 16 from 0.65 M (buckets up to 1024) or 1 M (2048) on, where there is no ragged tile, whose chain is longer
//                                   1 M, K = 16, bucket 128: 16.5 / 22.6; 0.7 M, K = 12, bucket 512: 13.5 / 15.2;
//                                   0.4 M, K = 12: 13.0 / 12.4; 1 M, K = 16, bucket 2048: 18.9 / 22.8; 0.7 M, K = 9,
//                                   2048: 14.7 / 13.5; 1 M, K = 32, bucket 128: 47.5 / 37.6; ragged, 1 M, K = 16,
//                                   bucket 512: 22.4 / 21.5, with a center 25.2 / 21.2
//     up to 2 with 4096 and 8192    0.5 M, K = 1, bucket 8192: 5.7 / 6.9; 0.2 M, K = 8, 4096: 11.8 / 8.1
//     none with 16384               0.5 M, K = 1: 9.3 / 8.3; 20 K, K = 1: 8.7 / 7.0; 0.5 M, K = 2: 12.8 / 8.5
// Buckets of 32768 would need 300 registers per lane.
// A wave that owns one chunk of every worker (buckets up to 4096, and wide ones) falls behind two launches where a
// round no longer fits about 1.2 GB, unless the workers' side is the dearer for it: level widths of 8 and more, whose
// codes cost the most to read back, or a center.  K = 16, 25 M, bucket 512: s = 4 415 / 388 us, s = 16 443 / 425, with a
// center 426 / 482; s = 65536 577 / 634; bucket 4096, s = 256 465 / 492, with a center 484 / 600; one bucket, 138 M,
// K = 4, s = 16 1298 / 1235.
inline bool round_fused_pays(const Shape& sh, uint32_t K, bool center) {
    const bool wide = sh.N > 32768, narrow = sh.N <= 4096 && sh.m < 8 && !center;
    if ((wide || narrow) && 4u * (uint64_t)K * sh.d + update_bytes(sh, K) > (1250ull << 20)) return false;
    if (sh.d >= (3u << 19)) return true;
    const uint64_t tile = sh.N <= 1024 ? 1024 : sh.N;
    if (sh.N <= 2048 && K <= 16 && sh.d >= (sh.N <= 1024 ? 5u << 17 : 15u << 16) && sh.d % tile == 0) return true;
    return K <= (sh.N <= 2048 || wide ? 8u : sh.N <= 8192 ? 2u : 0u);
}
int launch_round_fused(const Shape& sh, const QuantizeArgs& a, const AggregateArgs& g);
int launch_apply_update(const float* w, const float* zbar, float* u, float* zsum, uint64_t d,
                        hipStream_t stream);

int launch_quantize_fixed(const float* x, const float* center, uint64_t d, float delta, uint32_t b,
                          uint64_t seed, uint32_t round, uint32_t worker, void* codes, hipStream_t stream);
int launch_dequantize_fixed_update(const void* codes, uint64_t d, float delta, uint32_t b, const float* w,
                                   float* z, float* u, float* zsum, hipStream_t stream);
int launch_epoch_commit(float* w, float* zsum, uint32_t rounds, uint64_t d, hipStream_t stream);

void set_last_hip_error(int e);

}  // namespace qesgd
