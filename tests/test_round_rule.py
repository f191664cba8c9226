"""Which rounds take one launch (the rule that qesgd_round and qesgd_gradient_round share), asked on the host: measured shapes
get the side that was faster by more than the scatter, and the GPU tests of one launch against two do reach one launch."""
from paper_1901_03040_amd import binding as B
from test_built_kernels import host_values
from test_gpu_round_routes import LINES

WHOLE = 1 << 40


def routes(tmp_path, shapes, rule="round_chunks"):
    """What the rule says for each (d, K, bucket, s, center); round_chunks: 0 (two launches), 1 or 2 (chunks of a wave)."""
    body = "Shape sh{};\n"
    for d, K, bucket, s, center in shapes:
        lay = B.qesgd_layout_query(d, s, bucket)
        size = min(bucket, d)
        log2n = max(3, (size - 1).bit_length())
        body += (f"sh.d = {d}ull; sh.s = {s}; sh.m = {lay.level_bits}; sh.B = {size}ull; sh.nb = {lay.n_buckets}ull; sh.N = {1 << log2n}ull; "
                 f"sh.log2N = {log2n}; sh.lay.payload_bytes = {lay.payload_bytes}ull; "
                 f'std::printf("%u\\n", (unsigned){rule}(sh, {K}, {str(center).lower()}));\n')
    return [int(v) for v in host_values(tmp_path, body).split()]


# d, K, bucket, s, center; microseconds of two launches, of one; chunks.  Two sets of buffers in turn.
MEASURED = [
    (256, 6, 512, 4, False, 8.2, 7.8, 1), (30_000, 5, 2048, 4, False, 8.1, 7.9, 1), (256, 6, 256, 128, True, 8.5, 9.7, 0), (256, 4, 128, 256, False, 8.4, 6.2, 1),
    (47_104, 8, 128, 4, False, 7.7, 7.4, 1), (47_105, 8, 128, 4, False, 7.7, 8.7, 0), (207_884, 3, 4096, 16, False, 11.6, 6.8, 1),
    (8192, 2, 8192, 256, False, 9.0, 6.2, 2), (1_409_024, 3, 8192, 128, False, 14.6, 11.3, 2), (1_644_766, 16, 8192, 32, False, 37.7, 48.7, 0),
    (2_400_000, 1, 8192, 256, False, 13.9, 12.7, 2), (50_000_000, 4, 8192, 256, False, 366, 341, 2), (50_000_000, 16, 8192, 4, False, 800, 761, 2),
    (50_000_000, 8, 8192, 16, False, 502, 478, 2), (25_600_000, 8, 8192, 256, False, 323, 300, 2), (25_600_000, 2, 8192, 128, False, 132, 121, 2),
    (5_251_072, 24, 8192, 256, True, 169, 137, 2), (34_375_000, 32, 8192, 8, True, 1453, 1127, 2), (49_446_912, 6, 8192, 4, True, 450, 405, 2),
    (76_942_572, 4, 8192, 16, True, 575, 532, 2), (8_000_000, 16, 16_384, 4, False, 133.9, 122.0, 2), (1_899_695, 2, 16_384, 64, False, 16.5, 24.0, 0),
    (3_596_876, 24, 16_384, 65_536, False, 133.8, 94.0, 2), (3_937_603, 10, 16_384, 256, False, 61.0, 46.4, 2),
    (2_784_428, 5, 16_384, 64, False, 28.3, 32.4, 0), (1_458_272, 2, 16_384, 64, False, 14.2, 20.3, 0), (1_108_663, 1, 16_384, 128, False, 9.9, 13.9, 0),
    (698_105, 8, 2048, 16, True, 12.7, 14.9, 0), (1_500_000, 8, 4096, 256, False, 19.2, 16.7, 1), (25_000_000, 2, 512, 16, False, 122, 109, 1),
    (25_000_000, 16, 512, 256, False, 503, 467, 2), (30_638_080, 8, 16_384, 4, False, 292, 301, 0),
    (720_896, 16, WHOLE, 64, False, 30.9, 25.0, 1), (847_173, 32, 131_072, 256, False, 53.1, 65.0, 0), (216_470, 8, 131_072, 4, False, 11.2, 13.5, 0),
    (58_353_453, 16, 131_072, 32, True, 2526, 2097, 1), (138_357_544, 4, WHOLE, 16, False, 1244, 1320, 0)]


def test_measured_shapes_take_the_faster_side(tmp_path):
    for *_, two, one, chunks in MEASURED:
        assert (one < two) == (chunks > 0)
    got = routes(tmp_path, [m[:5] for m in MEASURED])
    assert {m[:5]: r for m, r in zip(MEASURED, got)} == {m[:5]: m[7] for m in MEASURED}


def test_gpu_tests_of_the_lines_lie_on_both_sides(tmp_path):
    got = routes(tmp_path, [(d, K, bucket, s, form == "center") for d, bucket, s, K, form, _ in LINES])
    assert [c[:5] + (r,) for c, r in zip(LINES, got)] == LINES


def test_policy_of_the_general_kernels_codes(tmp_path):
    """The ordinary one up to 288 MiB with power-of-two buckets and no center, otherwise up to 160 MiB."""
    shapes = [(20_588_235, 4, 2048, 65536, False), (60_000_000, 4, 256, 256, False), (37_777_777, 8, 2048, 256, False),
              (48_888_888, 4, 2048, 256, True), (38_888_888, 4, 3424, 256, False), (19_000_000, 4, 3424, 256, True)]
    assert routes(tmp_path, shapes, "general_codes_cached") == [1, 1, 0, 0, 0, 1]
