// Launches of a whole round: the scales of wide buckets where there are any, then the round (qesgd_round_device.h).
#include "qesgd_round.h"

namespace qesgd {

bool round_fused_covers(const Shape& sh, uint32_t norm_kind) {
    if (dense_wide(sh, norm_kind)) return true;
    return norm_kind == QESGD_NORM_L2 && sh.N == sh.B && sh.log2N >= 5 && sh.N <= 16384;
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
    uint64_t blocks;
    uint32_t chunks = 0;
    if (sh.N > kMaxSinglePassBucket) {
        const int rc = launch_dense_norms(p, sh, a);
        if (rc != QESGD_OK) return rc;
        p.xcd_group = xcd_group_log2(kWideWaves * kChunk);
        blocks = (sh.d + kWideWaves * kChunk - 1) / (kWideWaves * kChunk);
    } else {
        chunks = round_chunks(sh, a.K, a.center != nullptr);
        const uint64_t tile = round_tile(sh.N, chunks);
        blocks = (sh.nb * sh.N + tile - 1) / tile;
        p.full_tiles = (uint32_t)(sh.d / tile);
        p.tail_tiles = (uint32_t)(blocks - p.full_tiles);
        p.xcd_group = xcd_group_log2(tile);
    }
    if (blocks >= (1ull << 31)) return QESGD_ERR_DIM;
    switch (sh.m) {
        case 1: launch_round<1>(r, chunks, (uint32_t)blocks, a.stream); break;
        case 2: launch_round<2>(r, chunks, (uint32_t)blocks, a.stream); break;
        case 3: launch_round<3>(r, chunks, (uint32_t)blocks, a.stream); break;
        case 4: launch_round<4>(r, chunks, (uint32_t)blocks, a.stream); break;
        case 5: launch_round<5>(r, chunks, (uint32_t)blocks, a.stream); break;
        case 6: launch_round<6>(r, chunks, (uint32_t)blocks, a.stream); break;
        case 7: launch_round<7>(r, chunks, (uint32_t)blocks, a.stream); break;
        case 8: launch_round<8>(r, chunks, (uint32_t)blocks, a.stream); break;
        default: launch_round<16>(r, chunks, (uint32_t)blocks, a.stream); break;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_last_hip_error((int)e);
        return QESGD_ERR_HIP;
    }
    return QESGD_OK;
}

}  // namespace qesgd
