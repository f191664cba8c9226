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
constexpr uint64_t kSixWaveInput = 320ull << 20;        // from here on the quantiser's streams are held to six waves per SIMD:
constexpr uint64_t kSixWaveCodes = 48ull << 20;         // the vectors, or the packed blocks
constexpr uint64_t kCachedRaggedBytes = 144ull << 20;   // of the quantiser's ragged waves, the codes and the center (see quantize_params)
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

// LDS that a workgroup of `waves` waves, which has `fixed` bytes of its own, asks for besides so that a CU (160 KiB, handed out in
// steps of 1280 bytes; four SIMDs) takes 24 waves and no more: six per SIMD, whatever its registers allow.  0 where workgroups of
// that size cannot make 24.  (As amdgpu_waves_per_eu this would hold for every launch, and the compiler drops that attribute
// without a word where its lower bound is below what the workgroup's size implies.)
constexpr uint32_t kLdsBytes = 160u << 10, kLdsStep = 1280;
inline uint32_t six_wave_lds(uint32_t waves, uint32_t fixed) {
    if (24u % waves != 0u) return 0;
    const uint32_t share = kLdsBytes / (24u / waves) / kLdsStep * kLdsStep;
    return share > fixed ? share - fixed : 0u;
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
// power-of-two bucket of 32..16384 coordinates, L2 scale; or, behind the launches that find the scales, a dense
// wide bucket with the L2 scale.
bool round_fused_covers(const Shape& sh, uint32_t norm_kind);
// Tile of the one-launch round for buckets up to 16384.
inline uint64_t round_tile(uint64_t N, uint32_t chunks) { return N > 2u * chunks * kChunk ? N : 2u * chunks * kChunk; }
// One launch or two, and the chunks per wave of the one: 0 two launches, else 1 or 2 (always 2 from 8192 on; the
// wide buckets' kernel has 1).  One launch takes the workers of a tile one after the other, about 1 us each (2.4 us with
// buckets of 4096 and more, whose waves meet at a barrier per worker), which only a chip full of tiles hides; two
// launches spread tiles and workers over the chip at once, and read the codes back.  Two sets of buffers in turn, us,
// two launches / one.  "Bytes" are the K vectors', the packed blocks' and the update's; "odd" level widths are 3, 5, 6, 7,
// which the two launches store and read the dearest.
//   wide: up to 1250 MiB (138 M, K = 4, s = 16 1244 / 1320), from 1.5 M coordinates or up to 8 workers
//   8192 and 16384, whose chain is the longest
//     one generation of workgroups, K = 1, 2   0.5 M, K = 1, 8192 6.9 / 5.7; 1.5 M, K = 2, 8192 11.4 / 9.5; 2.4 M, K = 2,
//                               16384 16.8 / 14.6; but 5000, K = 2, 8192 8.6 / 8.8; 1.5 M, 16384 11.6 / 13.7
//     8 bits and more, K >= 8 from 8 M on, K >= 5 from 40 M on (K >= 16 with z_acc)   8 M, K = 8, 8192 89 / 81; 25 M, K = 16, 16384 480 / 468;
//                               5 M, K = 8 56 / 56; but 25 M, K = 4 171 / 171; 12 M, K = 8, 16384, z_acc 143 / 145
//     4 bits, K >= 16, 8192, from 20 M on      25 M 435 / 412; but 16384 430 / 443
//     odd, K >= 4, from 10 M on (8192 alone with z_acc)   12 M, K = 8, s = 128 137 / 124; 25 M, K = 4, s = 32, 16384 185 / 175;
//                               but 5 M, K = 4, s = 32 36 / 41; 25 M, K = 8, s = 32, 16384, z_acc 320 / 346
//     center, K >= 8 (8 bits, 8192: K >= 4), from 8 M on   12 M, K = 16, s = 4 231 / 203; 12 M, K = 4, s = 256 96 / 90, s = 4 80 / 86
//   up to 4096, below 1.5 M
//     whole tiles, from 0.65 M on (2048, not odd: 0.98 M; 4096: odd alone), up to 16 workers
//                               0.65 M, K = 16, s = 32, 128 21.5 / 18.4; 1 M, K = 16, bucket 128 22.6 / 16.5; 0.7 M, K = 9,
//                               2048 13.5 / 14.7; 1 M, K = 32, bucket 128 37.6 / 47.5
//     up to 5 workers           256, K = 5, bucket 128 8.6 / 7.3; 0.1 M, K = 5, 2048 8.7 / 8.6, K = 6 8.8 / 9.5; 0.3 M, K = 8, 512 8.8 / 10.5
//     8 up to 1024 with whole tiles, not odd, no z_acc   47104, K = 8, s = 4, bucket 128 7.7 / 7.4, with a ragged tile 7.7 / 8.7
//     8 from 0.9 M, 12 from 1.25 M on   1 M, K = 8, 512 15.0 / 14.4, K = 12 18.1 / 19.2; 1.3 M, K = 12, 512 20.8 / 19.5
//     with 4096 2 workers, 4 from 0.9 M on   0.4 M, K = 4 8.5 / 9.5; 1 M, K = 4 11.5 / 9.7
//   up to 4096, from 1.5 M on
//     odd, but not K = 1, 2 beyond 1000 MiB   12 M, K = 8, s = 128, 512 133 / 115; 50 M, K = 16, s = 8, 512 935 / 845; 50 M, K = 2, s = 8 238 / 247
//     up to 950 MiB, 1250 with 1 and 2 bits, 1100 with a center   25 M, K = 2, s = 16 122 / 109; 12 M, K = 16, s = 4 184 / 177;
//                               25 M, K = 2, s = 256 126 / 127; 12 M, K = 16, s = 16 198 / 210
//     beyond, two chunks (one / two): from 8 bits on with K * m >= 32, with 4 bits from 12 workers on, and with a center
//                               25 M, K = 16, s = 256, 512 503 / 505 / 467; 50 M, K = 8, s = 256, 256 575 / 563 / 536; 25 M, K = 16,
//                               s = 16, 256 430 / 460 / 418; center, 25 M, K = 16, s = 256 617 / 521 / 485; but 25 M, K = 8, s = 16
//                               238 / 261 / 248; 50 M, K = 2, s = 256 242 / 254 / 249; 12 M, K = 8, s = 4 110 / 101 / 114
//     center with 1 and 2 bits: one chunk      25 M, K = 16, s = 4 509 / 449
inline uint32_t round_chunks(const Shape& sh, uint32_t K, bool center, bool z_acc) {
    const uint64_t bytes = 4u * (uint64_t)K * sh.d + update_bytes(sh, K), mib = bytes >> 20;
    const uint64_t M = 1000000;
    const bool odd = 32u % sh.m != 0u;
    if (sh.N > kMaxSinglePassBucket) return bytes <= (1250ull << 20) && (sh.d >= (3u << 19) || K <= 8) ? 1 : 0;
    if (sh.N > 4096) {
        const bool narrow = sh.N == 8192;
        bool pays;
        if (center) pays = sh.d >= 8 * M && (K >= 8 || (K >= 4 && sh.m >= 8 && narrow));
        else if (odd) pays = sh.d >= 10 * M && K >= 4 && (narrow || !z_acc);
        else if (sh.m >= 8) pays = sh.d >= 8 * M && K >= (z_acc ? 16u : sh.d >= 40 * M ? 5u : 8u);
        else pays = sh.m == 4 && sh.d >= 20 * M && K >= 16 && narrow;
        const bool one_generation = K <= 2 && sh.d <= 256u * sh.N && sh.d >= (narrow ? (K - 1u) * 650000u : 1800000u);
        return pays || one_generation ? 2 : 0;
    }
    if (sh.d < (3u << 19)) {
        const uint64_t tile = round_tile(sh.N, 1);
        if ((odd || sh.N <= 2048) && K <= 16 && sh.d % tile == 0 && sh.d >= (odd || sh.N <= 1024 ? 5u << 17 : 15u << 16)) return 1;
        if (sh.N == 4096) return K <= (sh.d < 900000 ? 2u : 4u) ? 1 : 0;
        if (sh.N <= 1024 && !odd && !z_acc && K <= 8 && sh.d % tile == 0) return 1;
        return K <= (sh.d < 900000 ? 5u : sh.d < 1250000 ? 8u : 12u) ? 1 : 0;
    }
    if (odd) return K <= 2 && mib > 1000 ? 0 : 1;
    if (mib <= (sh.m < 4 ? 1250u : center ? 1100u : 950u)) return 1;
    if (center) return sh.m < 4 ? 1 : 2;
    return sh.m >= 4 && K * sh.m >= (sh.m == 4 ? 48u : 32u) ? 2 : 0;
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
