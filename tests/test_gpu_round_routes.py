"""Rounds in one launch at the edges of the rule that sends them there, against the calls they stand for, bit for bit:
level widths that do not divide a word, gradient rounds of ordinary buckets, two chunks per wave, buckets of 8192 and 16384."""
import pytest
import torch

from test_gpu_gradient_round import gradient_forms, inputs
from test_gpu_parity import B  # noqa: F401
from test_gpu_round import assert_same, both_forms

pytestmark = pytest.mark.gpu


def check(B, d, bucket, s, K, form):
    slab, w, c, zsum0 = inputs(d, K)
    if form == "gradient":
        for a, b in zip(*gradient_forms(B, slab, d, s, bucket, 0, K, w, c, zsum0)):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    else:
        _, out = both_forms(B, slab, c * 1e-3 if form == "center" else None, d, s, bucket, 0, 99, 3, K, w, zsum0)
        assert_same(out)


@pytest.mark.parametrize("form", ["push", "center", "gradient"])
@pytest.mark.parametrize("s", [2, 8, 32, 64, 128, 256])
@pytest.mark.parametrize("log2n", range(5, 13))
def test_small_rounds(B, log2n, s, form):
    bucket = 1 << log2n
    tile = max(1024, bucket)
    for d in (2 * tile, tile + bucket + 37, tile - 5, 33):    # whole tiles, a ragged tail, less than a tile
        check(B, d, bucket, s, 2, form)


@pytest.mark.parametrize("d,bucket,s,K,form", [
    # two chunks per wave, beyond 950 MiB (1100 with a center): 16 M whole tiles and a ragged one, every tile size
    (16_000_003, 32, 256, 16, "push"), (16_000_000, 1024, 16, 16, "push"), (16_000_003, 2048, 256, 16, "center"),
    (16_000_003, 4096, 65536, 16, "gradient"), (16_001_025, 512, 16, 16, "gradient"), (11_500_001, 4096, 256, 16, "push"),
    # one chunk beyond it
    (16_000_003, 512, 4, 16, "center"), (16_000_003, 4096, 128, 16, "push"), (16_000_003, 512, 8, 16, "gradient"),
    # buckets of 8192 and 16384: one generation of workgroups, then from 8 M (10 M odd) coordinates on
    (1_000_003, 8192, 16, 1, "push"), (1_000_003, 8192, 32, 2, "gradient"), (2_400_001, 16384, 256, 2, "center"),
    (8_000_003, 8192, 256, 8, "push"), (8_000_003, 16384, 65536, 16, "gradient"), (8_000_003, 16384, 4, 8, "center"),
    (10_000_003, 8192, 8, 4, "gradient"), (10_000_003, 16384, 128, 4, "push"), (20_000_003, 8192, 16, 16, "push")])
def test_large_rounds(B, d, bucket, s, K, form):
    check(B, d, bucket, s, K, form)
