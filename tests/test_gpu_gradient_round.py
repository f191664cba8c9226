"""qesgd_gradient_round and the wide-bucket form of qesgd_round against the calls they stand for, bit for
bit: scales finished in the last pass (up to 512 partial sums per bucket) and by a launch of their own,
one bucket and several, ragged ends, every level width, one launch and two."""
import pytest
import torch

from test_gpu_parity import B  # noqa: F401
from test_gpu_round import assert_same, both_forms

pytestmark = pytest.mark.gpu

WHOLE = 1 << 40


def gradient_forms(B, slab, d, s, bucket, norm_kind, K, w, z0, zsum0):
    lay = B.qesgd_layout_query(d, s, bucket)
    wsb = B.qesgd_workspace_bytes(d, s, bucket, K)
    ws = torch.full((wsb // 4,), float("nan"), device="cuda") if wsb else None
    stride = slab.stride(0)
    out = []
    for fused in (False, True):
        packed = B.alloc_packed(lay, K).fill_(0xA5)
        step, u = (torch.full((d,), float("nan"), device="cuda") for _ in range(2))
        z, zsum = z0.clone(), None if zsum0 is None else zsum0.clone()
        if fused:
            B.qesgd_gradient_round(slab, stride, d, s, bucket, norm_kind, 5, 2, K, packed, packed.stride(0), w, step, z, u,
                                   zsum, workspace=ws)
        else:
            B.qesgd_quantize_pack_batched(slab, stride, None, d, s, bucket, norm_kind, 5, 2, K, packed, packed.stride(0), ws)
            B.qesgd_unpack_aggregate(packed, packed.stride(0), K, d, s, bucket, step)
            B.qesgd_apply_update(z, step, z, None, d)
            B.qesgd_apply_update(w, z, u, zsum, d)
        torch.cuda.synchronize()
        out.append([packed, step, z, u] + ([] if zsum is None else [zsum]))
    return out


def inputs(d, K):
    g = torch.Generator(device="cuda").manual_seed(d + K)
    slab = torch.randn(K, (d + 63) // 64 * 64, generator=g, device="cuda") * 1e-3
    return slab, *(torch.randn(d, generator=g, device="cuda") for _ in range(3))


@pytest.mark.parametrize("d,bucket,K,norm_kind", [
    (1000, 128, 3, 0), (70_001, 4096, 4, 0), (70_001, 3008, 5, 1),         # one pass
    (32_776, WHOLE, 1, 0), (150_001, 65_536, 4, 0), (150_001, 65_536, 4, 1),
    (200_000, 48_000, 3, 0), (853_018, WHOLE, 8, 0), (853_018, WHOLE, 9, 0),   # 9: two launches
    (2_097_152, WHOLE, 2, 0), (2_097_160, WHOLE, 2, 0), (6_000_003, 4_194_304, 9, 0)])
@pytest.mark.parametrize("s", [2, 8, 256])
def test_gradient_round_is_the_four_calls(B, d, bucket, K, norm_kind, s):
    slab, w, z0, zsum0 = inputs(d, K)
    for zs in (zsum0, None):
        for a, b in zip(*gradient_forms(B, slab, d, s, bucket, norm_kind, K, w, z0, zs)):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("d,bucket,K,s", [
    (20_000_003, WHOLE, 16, 16),                                 # beyond 1250 MiB, and its vectors beyond the ordinary policy
    (1_600_001, WHOLE, 64, 4), (300_004, 65_536, 64, 256),       # the most workers, one launch and two
    (28_675, 128, 64, 65536), (1_600_003, 128, 64, 65536)])
def test_gradient_round_of_many_workers(B, d, bucket, K, s):
    slab, w, z0, zsum0 = inputs(d, K)
    for a, b in zip(*gradient_forms(B, slab, d, s, bucket, 0, K, w, z0, zsum0)):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("s", [2, 4, 8, 16, 32, 64, 128, 256, 65536])
@pytest.mark.parametrize("d,bucket,K", [(40_001, WHOLE, 3), (131_072 * 2, 131_072, 8), (300_004, 65_536, 2),
                                        (2_100_001, WHOLE, 2)])
def test_wide_round_is_the_two_calls(B, s, d, bucket, K):
    slab, w, c, zsum0 = inputs(d, K)
    for center in (None, c * 1e-3):
        _, out = both_forms(B, slab, center, d, s, bucket, 0, 99, 3, K, w, zsum0)
        assert_same(out)
    _, out = both_forms(B, slab, None, d, s, bucket, 0, 99, 3, K, w, zsum0, with_zbar=False, with_zsum=False)
    assert_same(out)


def test_scales_outside_the_short_form(B):
    """Zero, tiny, huge and infinite workers next to an ordinary one: the choice is made per worker."""
    d, K = 100_003, 6
    slab, w, _, zsum0 = inputs(d, K)
    slab *= torch.tensor([1.0, 0.0, 1e-25, 1e25, 1.0, 1.0], device="cuda")[:, None]
    slab[4, 77] = float("inf")
    for a, b in zip(*gradient_forms(B, slab, d, 16, WHOLE, 0, K, w, w * 0.5, zsum0)):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


def test_argument_errors(B):
    f = B.lib().qesgd_gradient_round
    p = [0x10000 * (i + 1) for i in range(7)]

    def call(x=p[0], K=2, packed=p[1], w=p[2], step=p[3], z=p[4], u=p[5], zsum=p[6], s=4, d=4096):
        return f(x, d, d, s, 512, 0, 1, 0, K, packed, 1 << 20, None, 0, w, step, z, u, zsum, None)
    for name in ("x", "packed", "w", "step", "z", "u"):
        assert call(**{name: None}) == B.ERR_NULL, name
    for name in ("w", "step", "z", "u", "zsum"):
        assert call(**{name: 0x10004}) == B.ERR_ALIGN, name
    assert call(K=0) == B.ERR_WORKERS and call(s=3) == B.ERR_LEVELS and call(d=0) == B.ERR_DIM
