"""The quantiser of buckets that are no power of two, the max norm and the level widths 3, 5, 6 and 7, at the edges of
its waves: buckets that end inside, at and behind a wave of 1024 (2048 above 16384), a last bucket that ends anywhere in
one, a workgroup of several buckets, narrow buckets, and the last pass of wide ones.  Scales, code words and the bytes
behind them against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from test_gpu_parity import B  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,norm_kind,with_center", [(32, 1, False), (128, 0, True), (256, 0, False), (2, 1, True), (65536, 1, False)])
@pytest.mark.parametrize("bucket,last", [
    (544, 1), (1024, 1023), (1056, 33), (2016, 2015), (2080, 2049), (3008, 1030), (4096, 3071), (6176, 4099), (8192, 7),
    (12_000, 11_264), (16_416, 2047), (20_480, 18_437), (32_736, 30_721), (32_768, 4), (64, 63), (512, 511), (256, 5),
    (33_792, 1_025), (65_536, 4_097), (98_304, 65_535)])
def test_edges_of_waves(oracle, B, bucket, last, s, norm_kind, with_center):
    K, d = 3, 2 * bucket + last
    g = torch.Generator(device="cpu").manual_seed(bucket * 7 + s)
    stride = (d + 3) // 4 * 4
    x = torch.zeros(K, stride)
    x[:, :d] = torch.randn(K, d, generator=g) * 1e-2
    center = torch.randn(d, generator=g) * 1e-2 if with_center else None
    lay = B.qesgd_layout_query(d, s, bucket)
    wsb = B.qesgd_workspace_bytes(d, s, bucket, K)
    ws = torch.empty(wsb // 4, device="cuda") if wsb else None
    packed = B.alloc_packed(lay, K)
    packed.fill_(0xA5)
    B.qesgd_quantize_pack_batched(x.cuda(), stride, None if center is None else center.cuda(), d, s, bucket, norm_kind, 77, 5, K,
                                  packed, packed.stride(0), ws)
    torch.cuda.synchronize()
    for k in range(K):
        want = oracle.quantize_pack(x[k, :d].numpy(), s, bucket, 77, 5, k, center=None if center is None else center.numpy(),
                                    norm_kind=norm_kind)
        for got, w, what in zip(B.planes(packed[k], lay), want, ("scales", "signs", "levels")):
            assert np.array_equal(got.cpu().numpy().view(np.uint32), w.view(np.uint32)), (k, what)
        for end, upto in ((lay.norms_off + 4 * lay.n_buckets, lay.signs_off), (lay.signs_off + 4 * lay.sign_words, lay.levels_off),
                          (lay.levels_off + 4 * lay.level_words, lay.bytes_per_worker)):
            assert bool((packed[k, end:upto] == 0xA5).all()), (k, "a gap between planes was written")


@pytest.mark.parametrize("bucket,s,norm_kind,K,with_center", [
    (992, 4, 0, 3, True), (992, 256, 1, 3, False), (2016, 128, 0, 3, True), (2016, 65536, 0, 10, False), (3008, 65536, 1, 10, False),
    (5024, 16, 0, 3, True), (12_000, 32, 1, 3, True), (20_000, 8, 0, 3, True), (48_000, 64, 0, 3, False), (48_000, 4, 1, 3, True),
    (2048, 65536, 1, 10, False), (256, 65536, 1, 10, False), (2048, 65536, 1, 17, False)])     # 170 and 289 MiB of codes
def test_streams_beyond_the_caches(B, bucket, s, norm_kind, K, with_center):
    """More than 96 MiB of input (and with 10 workers 160 MiB of codes) against one call per worker, which stays below:
    the policy of the streams and the order of the workers change no bit."""
    d = 8_400_003
    g = torch.Generator(device="cuda").manual_seed(bucket + s)
    stride = (d + 3) // 4 * 4
    x = torch.randn(K, stride, generator=g, device="cuda") * 1e-2
    center = torch.randn(d, generator=g, device="cuda") * 1e-2 if with_center else None
    lay = B.qesgd_layout_query(d, s, bucket)
    wsb = B.qesgd_workspace_bytes(d, s, bucket, K)
    ws = torch.empty(wsb // 4, device="cuda") if wsb else None
    packed, want = B.alloc_packed(lay, K).fill_(0xA5), B.alloc_packed(lay, K).fill_(0xA5)
    B.qesgd_quantize_pack_batched(x, stride, center, d, s, bucket, norm_kind, 77, 5, K, packed, packed.stride(0), ws)
    for k in range(K):
        B.qesgd_quantize_pack(x[k], center, d, s, bucket, norm_kind, 77, 5, k, want[k], ws)
    assert torch.equal(packed, want)
