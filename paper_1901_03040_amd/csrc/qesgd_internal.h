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
constexpr uint64_t kCachedGeneralCodeBytes = 288ull << 20;   // of the packed blocks, for the general kernels (see general_codes_cached)
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

// The general kernels' codes of power-of-two buckets (the max norm; odd level widths are indifferent) are better written with the
// ordinary policy as far as the memory-side cache holds part of them for the server's call.  Whole two-call round, max norm,
// non-temporal / ordinary, us: K = 4, s = 65536, 20.6 M (167 MiB) 175 / 166, 31.8 M (257) 271 / 254; K = 4, s = 256, 38.9 M (167)
// 282 / 273, 60 M (257) 438 / 415; K = 8, s = 256, 37.8 M (324) 427 / 439, 50 M (429) 566 / 593.  With a center, and in buckets that are
// no power of two, the other one is (K = 4, s = 256, center, 48.9 M 390 / 409; 3424, 38.9 M 277 / 280, 60 M 435 / 440).
inline bool general_codes_cached(const Shape& sh, uint32_t K, bool center) {
    return K * sh.lay.payload_bytes <= (!center && sh.N == sh.B ? kCachedGeneralCodeBytes : kCachedCodeBytes);
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
// One launch or two, and the chunks per wave of the one: 0 two launches, else 1 or 2 (always 2 from 8192 on; the wide buckets'
// kernel has 1).  One launch takes the workers of a tile one after the other, which only a chip full of tiles hides; two
// launches spread tiles and workers over the chip at once, and read the codes back.  Drawn from 18000 shapes timed both ways
// (d = 256 .. 60 M, K = 1 .. 32, all level widths, two sets of buffers in turn), where it takes 0.4% more than always the better
// side; microseconds, two launches / one.  "Dear" level widths are 3, 5, 6, 7 and those of 8 bits and more, whose codes cost
// the most to read back.
//   8192 and 16384: a workgroup of 8 or 16 waves fills a CU, so 256 tiles are one generation, and it takes as long however few
//   tiles it has.
//     one generation, full enough for its workers   1.4 M, K = 3, s = 128, 8192 14.6 / 11.3; 3.6 M, K = 24, s = 65536, 16384 133.8 / 94.0;
//                                  but 1.9 M, K = 2, s = 64, 16384 16.5 / 24.0; 1.6 M, K = 16, s = 32, 8192 37.7 / 48.7
//     more, K >= 4, where a last one of up to four is half full, and the codes or the workers are many: dear, a center, 10 workers
//     with 16384, beyond 2000 MiB  5.3 M, K = 24, s = 256, center, 8192 169 / 137; 8 M, K = 16, s = 4, 16384 134 / 122; 50 M, K = 16, s = 4,
//                                  8192 800 / 761; 34 M, K = 32, s = 8, center, 8192 1453 / 1127; 50 M, K = 4, s = 256, 8192 366 / 341; but 31 M, K = 8,
//                                  s = 4, 16384 292 / 301
//   up to 4096, short vectors: the chain of K workers, at the ragged tile if there is one, against one launch more at first (8 us
//   for two calls' worth of host work), then against what two launches take for the bytes, which grows with K too: the line
//   rises with d, measured as a square.  One launch up to 0.3 M, K = 3 .. 8: bucket 128 .. 512, ragged 5.5 6.1 7.1 7.8 8.8 9.3, whole 5.4 5.2
//   5.7 6.2 6.9 7.3; 4096, ragged 6.7 7.2 8.7 9.9 10.7 12.1; widths 3, 5, 6, 7 and 16 and a center add 0.5 to 2
//                                  0.2 M, K = 3, 4096 11.6 / 6.8; 1 M, K = 8, 512 15.0 / 14.4; 47 K, K = 8, s = 4, 128, one ragged 7.7 / 8.7
//     and by the bytes of the K vectors, the packed blocks and the update   25 M, K = 2, s = 16 122 / 109, s = 256 126 / 127; 12 M,
//                                  K = 16, s = 16 198 / 210; 50 M, K = 16, s = 8 935 / 845, K = 2 238 / 247
//     beyond, two chunks (one / two): from 8 bits on with K * m >= 32, with 4 bits from 12 workers on, and with a center
//                                  25 M, K = 16, s = 256, 512 503 / 505 / 467; 25 M, K = 16, s = 16, 256 430 / 460 / 418; but
//                                  25 M, K = 8, s = 16 238 / 261 / 248; 12 M, K = 8, s = 4 110 / 101 / 114
//   wide: up to 1250 MiB, beyond it with widths 3, 5, 6, 7 or a center   138 M, K = 4, s = 16 1244 / 1320; 58 M, K = 16, s = 32, center
//                                  2526 / 2097; many workers from 0.55 M coordinates on (more than 16, one tile ragged: 1.5 M)
//                                  0.72 M, K = 16, s = 64 30.8 / 25.0; 0.85 M, K = 32, s = 256 53 / 65; 216 K, K = 8, s = 4 11.2 / 13.5
inline uint32_t round_chunks(const Shape& sh, uint32_t K, bool center) {
    const uint64_t mib = (4u * (uint64_t)K * sh.d + update_bytes(sh, K)) >> 20;
    const bool odd = 32u % sh.m != 0u, dear = odd || sh.m >= 8;
    if (sh.N > kMaxSinglePassBucket) {
        const bool whole = sh.d % 2048u == 0u;
        if (mib >= 1250 && !center && !odd) return 0;
        if (K <= (whole ? 8u : 7u)) return 1;
        return sh.d >= (whole || K <= 16 ? 550000u : 3u << 19) ? 1 : 0;
    }
    if (sh.N > 4096) {
        const uint64_t tiles = (sh.d + sh.N - 1) / sh.N, generations = (tiles + 255u) / 256u, idle = 256u * generations - tiles;
        const bool few8 = sh.N == 8192 && K <= 2;
        if (generations == 1) {
            uint32_t need = sh.N == 8192 ? 55u + 24u * K : 100u + 12u * K;
            const uint32_t most = sh.N == 8192 ? (sh.m >= 8 ? 220u : 257u) : sh.m >= 8 ? 150u : 190u;
            if (need > most || (sh.N == 16384 && odd && K >= 3)) need = most;
            if (few8 && (K == 1 || sh.d % sh.N == 0u)) need = 0;
            return tiles >= need ? 2 : 0;
        }
        if (few8 && generations == 2) return K == 1 || idle <= 128u ? 2 : 0;
        if (generations > 4 && odd) return 2;
        const bool heavy = dear || (center && (K >= 6 || mib > 1400)) || (sh.N == 16384 && K >= 10) ||
                           (mib > 2000 && sh.m > 1 && K * sh.m >= (sh.N == 8192 ? 12u : 32u));
        return K >= 4 && heavy && (generations > 4 || idle <= 128u) ? 2 : 0;
    }
    if (sh.d < 3000000u) {
        const bool whole = sh.d % round_tile(sh.N, 1) == 0u;
        const double M = (double)sh.d * 1e-6, M2 = M * M;
        double most;
        if (whole) {
            most = (sh.N <= 1024 ? 8.5 : sh.N == 2048 ? 6.5 : 4.8) + (sh.N == 4096 ? 12.0 : 20.0) * M2;
        } else {
            most = (sh.N <= 512 ? 6.0 : sh.N == 1024 ? 5.6 : sh.N == 2048 ? 5.0 : 4.2) - (odd || sh.m == 16 ? 0.5 : 0.0) + (sh.N == 4096 ? 3.5 : 7.0) * M2;
            if (center) most *= 0.9;
        }
        if (K > most) return 0;
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
