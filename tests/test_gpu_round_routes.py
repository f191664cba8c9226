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


WHOLE = 1 << 40
# Just on either side of each line of the rule: d, bucket, s, K, form, route (0 two launches, else the chunks of a wave in the one)
LINES = [
    # up to 4096, by workers and length, ragged and whole tiles
    (377_003, 512, 4, 7, "push", 0), (379_003, 512, 4, 7, "push", 1), (273_408, 512, 256, 10, "center", 0), (274_432, 512, 256, 10, "center", 1),
    (1_034_003, 2048, 8, 12, "gradient", 0), (1_036_003, 2048, 8, 12, "gradient", 1), (503_003, 128, 256, 7, "center", 0), (505_003, 128, 256, 7, "center", 1),
    (358_003, 1024, 65536, 6, "push", 0), (360_003, 1024, 65536, 6, "push", 1), (688_128, 2048, 16, 16, "push", 0), (690_176, 2048, 16, 16, "push", 1),
    (1_041_003, 4096, 2, 8, "push", 0), (1_043_003, 4096, 2, 8, "push", 1), (315_392, 4096, 64, 6, "gradient", 0), (319_488, 4096, 64, 6, "gradient", 1),
    (2_999_999, 4096, 2, 64, "push", 0), (3_000_001, 4096, 2, 64, "push", 1),
    # 8192: one generation of workgroups, two, more; beyond 2000 MiB
    (8192, 8192, 256, 2, "push", 2), (8193, 8192, 256, 2, "push", 0), (835_584, 8192, 32, 3, "center", 0), (835_585, 8192, 16, 2, "gradient", 2),
    (1_032_192, 8192, 128, 3, "push", 0), (1_032_193, 8192, 128, 3, "push", 2), (1_794_048, 8192, 65536, 16, "gradient", 0),
    (1_794_053, 8192, 65536, 16, "gradient", 2), (2_097_152, 8192, 16, 16, "push", 0), (2_097_153, 8192, 256, 1, "center", 2), (4_194_305, 8192, 256, 1, "push", 0),
    (3_137_536, 8192, 16, 2, "push", 0), (3_137_537, 8192, 16, 2, "push", 2), (3_137_536, 8192, 256, 4, "gradient", 0), (3_137_537, 8192, 256, 4, "gradient", 2),
    (8_388_608, 8192, 8, 1, "push", 0), (8_388_609, 8192, 8, 1, "push", 2), (8_388_609, 8192, 4, 5, "center", 0), (8_388_609, 8192, 4, 6, "center", 2),
    (36_500_003, 8192, 16, 8, "push", 0), (37_000_003, 8192, 16, 8, "push", 2),
    # 16384
    (2_015_232, 16384, 8, 2, "gradient", 0), (2_015_233, 16384, 8, 2, "gradient", 2), (2_441_216, 16384, 256, 5, "push", 0), (2_441_217, 16384, 256, 5, "push", 2),
    (3_096_576, 16384, 4, 8, "center", 0), (3_096_577, 16384, 4, 8, "center", 2), (6_275_072, 16384, 4, 10, "push", 0), (6_275_073, 16384, 4, 10, "push", 2),
    (6_291_456, 16384, 4, 9, "push", 0), (10_485_760, 16384, 128, 4, "gradient", 2),
    (38_000_003, 8192, 16, 4, "center", 0), (39_000_003, 8192, 16, 4, "center", 2),
    # wide, by workers and length, beyond 1250 MiB
    (40_001, WHOLE, 4, 7, "push", 1), (40_001, WHOLE, 4, 8, "push", 0), (40_960, WHOLE, 16, 8, "gradient", 1), (40_960, WHOLE, 16, 9, "gradient", 0),
    (549_999, 65536, 32, 16, "center", 0), (550_001, 65536, 32, 16, "center", 1), (550_001, 65536, 32, 17, "center", 0), (1_572_864, 65536, 32, 17, "push", 1),
    (20_000_003, WHOLE, 16, 16, "push", 0), (20_000_003, WHOLE, 16, 16, "center", 1), (20_000_003, WHOLE, 8, 16, "gradient", 1),
    # up to 4096, by bytes: 950, 1000, 1100 and 1250 MiB
    (10_000_003, 512, 16, 16, "push", 1), (11_300_003, 512, 16, 16, "push", 2), (11_000_003, 1024, 256, 16, "center", 1), (11_500_003, 1024, 256, 16, "center", 2),
    (30_000_003, 128, 8, 2, "push", 1), (38_000_003, 128, 8, 2, "push", 0), (14_000_003, 2048, 4, 16, "push", 1), (16_500_003, 2048, 4, 16, "push", 0),
    (16_500_003, 2048, 4, 16, "center", 1)]


@pytest.mark.parametrize("d,bucket,s,K,form,route", LINES)
def test_both_sides_of_each_line(B, d, bucket, s, K, form, route):
    check(B, d, bucket, s, K, form)
