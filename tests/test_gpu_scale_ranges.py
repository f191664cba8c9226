"""Where the quantiser's arithmetic and tile order change form: bucket norms at and beyond the ends of
the range in which the scale is folded into one multiplication, coordinates that carry their whole
bucket (the level that must not overflow), negative zeros, and vectors long enough that tiles are
dealt to the XCDs in groups, with tiles left over."""
import numpy as np
import pytest
import torch

from test_gpu_shapes import B, run_and_compare  # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

# target norms: underflow of the squares, both edges of each range test (2^-60, 2^60; totals 2^-90,
# 2^120), ordinary, overflow of the squares
EXPONENTS = [-149, -130, -75, -61, -60, -59, -46, -45, -44, -8, 0, 59, 60, 61, 63, 64, 100]


def bucket_values(g, bucket, form):
    v = torch.randn(bucket, generator=g, dtype=torch.float64)
    if form == 1:                                   # one coordinate is the whole bucket
        v = torch.zeros(bucket, dtype=torch.float64)
        v[int(torch.randint(bucket, (1,), generator=g))] = -1.0 if bucket % 64 else 1.0
    elif form == 2:                                 # nearly: everything else is tiny
        v = v * 1e-7
        v[3] = 1.0 + float(torch.rand(1, generator=g))
    elif form == 3:                                 # signed zeros
        v = torch.where(torch.rand(bucket, generator=g) < 0.5, v * 0.0, v)
    return v / v.norm()


@pytest.mark.parametrize("bucket", [32, 96, 512, 4096, 8192])
@pytest.mark.parametrize("s", [2, 4, 8, 16, 32, 64, 128, 256, 65536])
def test_norms_across_the_exponent_range(oracle, B, s, bucket):
    g = torch.Generator(device="cpu").manual_seed(s + bucket)
    parts = [torch.zeros(bucket, dtype=torch.float64)]
    for e in EXPONENTS:
        for form in range(4):
            parts.append(bucket_values(g, bucket, form) * 2.0 ** e)
    parts.append(-torch.zeros(bucket, dtype=torch.float64))
    x = torch.cat(parts).float()
    assert torch.isfinite(x).all()
    run_and_compare(oracle, B, x.cuda(), s, bucket, 11, 2)


@pytest.mark.parametrize("s", [2, 4, 16, 256])
@pytest.mark.parametrize("bucket", [512, 4096])
@pytest.mark.parametrize("tail", [0, 3 * 8192 + 40])
@pytest.mark.parametrize("centered", [False, True])
def test_tiles_dealt_in_groups(oracle, B, s, bucket, tail, centered):
    d, K = 2 * (1 << 19) + tail, 3                  # two rounds of eight 64 K-coordinate groups
    g = torch.Generator(device="cpu").manual_seed(d + s)
    x = (torch.randn(K, d, generator=g) * 1e-3).cuda()
    center = (torch.randn(d, generator=g) * 1e-3).cuda() if centered else None
    run_and_compare(oracle, B, x, s, bucket, 4, 9, K=K, center=center)


@pytest.mark.parametrize("bucket,d", [(96, 4000), (3008, 20_000), (4096, 16_384), (65_536, 200_000)])
@pytest.mark.parametrize("s", [2, 8, 16, 256, 65536])
def test_nan_and_infinity_keep_the_formula(oracle, B, s, bucket, d):
    """A maximum passes over a NaN, so the scale stays finite: the level is the minimum's other operand,
    s - 1, with the sign bit of no number, 0.  Infinities make the scale infinite under either norm."""
    g = torch.Generator(device="cpu").manual_seed(s + d)
    for norm in (0, 1):
        for odd in (float("nan"), -float("nan"), float("inf"), -float("inf")):
            x = torch.randn(d, generator=g) * 1e-2
            x[torch.randint(d, (5,), generator=g)] = odd
            lay = B.qesgd_layout_query(d, s, bucket)
            packed = B.alloc_packed(lay, 1).zero_()
            wsb = B.qesgd_workspace_bytes(d, s, bucket, 1)
            ws = torch.empty(wsb // 4, device="cuda") if wsb else None
            B.qesgd_quantize_pack(x.cuda(), None, d, s, bucket, norm, 3, 1, 0, packed[0], ws)
            n, sg, lv = (t.cpu().numpy() for t in B.planes(packed[0], lay))
            on, osw, olw = oracle.quantize_pack(x.numpy(), s, bucket, 3, 1, 0, norm_kind=norm)
            assert np.array_equal(n, on, equal_nan=True), (norm, odd, "norms")
            assert np.array_equal(sg.view(np.uint32), osw), (norm, odd, "signs")
            assert np.array_equal(lv.view(np.uint32), olw), (norm, odd, "levels")
