// What the unit that chooses a round's launches and those that hold its kernels share (not installed).
#pragma once

#include "qesgd_quantize_device.h"

namespace qesgd {

struct RParams {
    QParams q;
    const float* w;
    float* zbar;
    float* u;
    float* zsum;
    float* z_acc;    // nullable: z_acc += the mean
    float rcpK;      // exact 1/K when K is a power of two, else 0
    uint32_t K;
};

// Queues the round's last launch for level width M: chunks of a wave (0: the wide buckets' kernel), workgroups.
// Defined in qesgd_round_device.h and instantiated in qesgd_round_*.hip, a few widths each, since they take long to compile.
// A unit that sees the definition compiles every kernel of the widths it calls; only those six include it.
template <int M>
void launch_round(const RParams& r, uint32_t chunks, uint32_t blocks, hipStream_t st);

// Waves of a workgroup of the wide buckets' kernel.
constexpr uint32_t kWideWaves = 4;

}  // namespace qesgd
