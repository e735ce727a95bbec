"""How launches are cut (csrc/launch_rules.h), host code only: sizes that were timed on both sides of a rule go to the side that
was faster."""
import ctypes
import os

import pytest

from paper_2509_17396_amd import binding as ep
from paper_2509_17396_amd import build


@pytest.fixture(scope="module")
def rules():
    so = os.path.join(os.path.dirname(build.LIB), "selftest", "liblaunch_rules.so")
    if not os.path.exists(so):
        build.build_selftests()
    return ctypes.CDLL(so)


BF16, F32 = ep.DTYPE_BF16, ep.DTYPE_F32


# dtype, head_dim, rows per workgroup, heads, 64-key tiles; what pass 2 took with the fit's splits against the estimate's
@pytest.mark.parametrize("fitted,sizes", [
    # 1.14 to 1.32 times as long, 1.08 to 1.13, 1.10 to 1.21
    (False, [(BF16, 136, 128, 32, 204), (BF16, 136, 128, 224, 16), (BF16, 192, 128, 64, 204), (BF16, 256, 128, 64, 128),
             (F32, 72, 128, 64, 128), (F32, 96, 128, 32, 204), (F32, 128, 128, 64, 128),
             (BF16, 32, 32, 896, 16), (BF16, 32, 32, 512, 40), (BF16, 8, 32, 256, 128), (F32, 64, 64, 896, 64)]),
    # 0.83 on average, and forms between those that were timed
    (True, [(BF16, 32, 64, 64, 64), (BF16, 96, 128, 96, 16), (BF16, 128, 128, 896, 64), (BF16, 64, 256, 96, 64),
            (BF16, 136, 32, 32, 64), (BF16, 256, 64, 96, 64), (F32, 72, 64, 32, 64), (F32, 128, 32, 64, 16),
            (BF16, 40, 32, 224, 64), (BF16, 64, 192, 96, 128)])])
def test_key_splits_of_the_max_reduction(rules, fitted, sizes):
    for size in sizes:
        a, b = ctypes.c_int(0), ctypes.c_int(0)
        assert bool(rules.max_splits(*size, ctypes.byref(a), ctypes.byref(b))) == fitted, size
        assert 1 <= a.value <= 32 and 1 <= b.value <= 32


# heads, scores per head, kept rows, bytes of a row: one launch takes longer by 2 to 26 %, or is faster by 1 to 31 %
@pytest.mark.parametrize("one_launch,sizes", [
    (False, [(1024, 4096, 128, 16), (256, 8192, 512, 16), (512, 2049, 500, 16), (512, 4096, 256, 64), (512, 4096, 256, 128),
             (200, 8193, 600, 16), (256, 16384, 500, 16), (160, 16384, 1500, 64), (160, 4096, 1000, 16), (256, 4096, 1500, 16),
             (896, 8192, 140, 128), (1024, 300, 128, 16), (1024, 300, 128, 32), (384, 8192, 700, 32), (512, 16384, 200, 64),
             (512, 4096, 64, 64)]),
    (True, [(1, 16384, 130, 16), (8, 12000, 130, 16), (2, 4096, 4000, 16), (64, 16384, 256, 16), (96, 4096, 1300, 16),
            (100, 4096, 130, 16), (128, 4096, 1000, 16), (128, 8192, 200, 16), (128, 16384, 128, 16), (128, 16384, 1000, 128),
            (128, 2048, 1000, 16), (256, 1024, 512, 16), (512, 1024, 256, 64), (700, 1500, 300, 64), (256, 8192, 512, 128),
            (200, 8193, 600, 128), (256, 2100, 1000, 128), (160, 16384, 1500, 128), (32, 4096, 2048, 256), (64, 2024, 1024, 192),
            (1, 2, 1, 16)])])
def test_selection_and_compaction_in_one_launch_where_it_is_faster(rules, one_launch, sizes):
    for size in sizes:
        assert (rules.select_compact_parts(*size) > 0) == one_launch, size


def test_ranges_fit_a_workgroup(rules):
    """At most 32, one report bit each, and no more rows than 16 rounds of a workgroup move."""
    for heads in (1, 3, 32, 200, 4000):
        for n in (2, 2048, 2049, 16384, 16385):
            for kept in sorted({1, n // 3 + 1, n - 1}):
                for row in (16, 48, 192, 256, 512):
                    parts = rules.select_compact_parts(heads, n, kept, row)
                    assert 0 <= parts <= 32 and (n <= 16384 or parts == 0)
                    if parts:
                        assert -(-kept // parts) <= 16 * ((512 if n <= 2048 else 1024) // (row // 16))


# queries, episodes: three centroids at a time took 0.7 to 0.97, or 1.02 to 1.27 times as long as two
@pytest.mark.parametrize("rows,sizes", [
    (3, [(1, 9), (1, 10), (256, 12), (1000, 9), (1000, 12), (1, 17), (1000, 20), (1000, 25), (256, 20), (1000, 24), (40, 32),
         (256, 64), (1000, 300)]),
    (2, [(1, 1), (256, 2), (1000, 3), (1000, 4), (40, 5), (1, 8), (1000, 8), (1, 13), (40, 14), (256, 16), (1000, 16), (1000, 17),
         (1000, 32), (1000, 64)])])
def test_centroids_at_a_time(rules, rows, sizes):
    for size in sizes:
        assert rules.match_rows(*size) == rows, size


# segments, clusters, dims: workgroups of 16 waves took 0.7 to 0.98, or 1.05 to 1.44 times as long as those of four
@pytest.mark.parametrize("threads,sizes", [
    (1024, [(1873, 10, 1024), (2, 1, 384), (100, 10, 1024), (4000, 24, 384), (4000, 2, 1536), (25600, 256, 384)]),
    (256, [(600, 300, 384), (8000, 1000, 100), (30000, 1000, 1024), (51200, 512, 384), (640, 10, 4096), (24000, 24, 4096),
           (1000, 1, 8192)])])
def test_waves_that_look_for_a_medoid(rules, threads, sizes):
    for size in sizes:
        per_cluster = ctypes.c_int(0)
        assert rules.medoid_shape(*size, ctypes.byref(per_cluster)) == threads, size
        assert 1 <= per_cluster.value <= max(1, 256 // size[1])


def test_any_number_of_segments_and_clusters(rules):
    for n in (1, 2, 1 << 20, (1 << 31) - 1):
        for clusters in (1, 255, 256, 257, 1 << 24, (1 << 31) - 1):
            for dim in (1, 2048, 2049, 8192):
                per_cluster = ctypes.c_int(0)
                rules.medoid_shape(n, clusters, dim, ctypes.byref(per_cluster))
                assert 1 <= per_cluster.value <= max(1, 256 // clusters)


def attention_shape(rules, heads, rows, n, d, causal=1, patch=64):
    rules.attention_shape.restype = ctypes.c_int64
    out = (ctypes.c_int * 4)()
    return rules.attention_shape(heads, rows, patch, n, causal, d, out), *out


def test_key_splits_of_the_attention_cover_the_keys(rules):
    for heads in (1, 3, 32, 200, 65535):
        for rows in (1, 33, 250, 1000, 16384):
            for n in (1, 64, 65, 1000, 4097, 1 << 20, 1 << 24):
                for d in (8, 40, 64, 72, 128):
                    for causal in (0, 1):
                        room, waves, groups, splits, each = attention_shape(rules, heads, rows, n, d, causal)
                        keys = n + 64 * causal
                        assert waves * groups <= 8 and 1 <= splits <= 64, (heads, rows, n, d)
                        if splits == 1:
                            assert each >= keys and room == 0
                            continue
                        assert each % 64 == 0 and (splits - 1) * each < keys <= splits * each, (heads, rows, n, d)
                        assert room == heads * splits * rows * (d + 2) * 4
                        # three rounds of workgroups of 256 rows at most
                        assert room <= 3 * 256 * 256 * (d + 2) * 4


# heads, rows, keys with the patch's, head_dim: the attention in key splits took 0.1 to 0.8, or 1.1 times and more as long as without
@pytest.mark.parametrize("split,sizes", [
    (True, [(2, 256, 18135, 128), (8, 192, 12008, 128), (16, 224, 11182, 128), (4, 128, 7303, 128), (30, 512, 11232, 128),
            (8, 64, 5724, 128), (4, 256, 16377, 64), (4, 64, 5439, 64)]),
    (False, [(216, 448, 4442, 128), (168, 256, 1146, 128), (16, 512, 842, 128), (72, 164, 1650, 128), (56, 128, 1949, 64),
             (40, 136, 6276, 64), (8, 107, 991, 64)])])
def test_attention_in_key_splits_where_it_is_faster(rules, split, sizes):
    for heads, rows, n, d in sizes:
        assert (attention_shape(rules, heads, rows, n, d, causal=0)[3] > 1) == split, (heads, rows, n, d)


# heads, rows, keys, head_dim: both scoring passes took 0.34 to 0.89 times as long with the workgroups of a head on all XCDs, or 1.02 times
# and more; heads that are a multiple of 8 stay on their own
@pytest.mark.parametrize("spread,sizes", [
    (1, [(1, 1792, 16000, 128), (1, 512, 4000, 128), (4, 512, 16000, 128), (12, 512, 16000, 128), (28, 512, 4000, 128), (12, 192, 4000, 128),
         (12, 192, 16000, 128), (28, 192, 4000, 128), (3, 400, 2500, 96)]),
    (0, [(28, 512, 700, 128), (12, 1792, 700, 128), (4, 512, 700, 128), (28, 64, 4000, 128), (44, 256, 864, 128), (22, 256, 7729, 64),
         (8, 512, 16000, 128), (16, 192, 16000, 128), (896, 192, 4096, 128)])])
def test_heads_on_all_xcds_where_that_is_faster(rules, spread, sizes):
    for size in sizes:
        assert rules.score_form(BF16, *size, ctypes.byref(ctypes.c_int(0))) == spread, size


# heads, rows, keys: the groups of waves that were fastest among 1, 2 and 4; 0 where pass 2 streams the keys
@pytest.mark.parametrize("groups,sizes", [
    (4, [(8, 1792, 700), (8, 512, 700), (1, 1792, 16000)]), (2, [(8, 1792, 4000), (8, 512, 4000)]), (1, [(8, 512, 16000), (128, 512, 8192)]),
    (0, [(8, 192, 4096), (128, 256, 8192)])])
def test_groups_of_the_key_stationary_pass(rules, groups, sizes):
    for size in sizes:
        got = ctypes.c_int(-1)
        rules.score_form(BF16, *size, 128, ctypes.byref(got))
        assert got.value == groups, size


def test_groups_fit_the_lds(rules):
    for heads in (1, 3, 8, 64):
        for rows in (257, 1024, 4096, 8192, 16384):
            for n in (1, 700, 8192, 100000):
                for d in (64, 128):
                    got = ctypes.c_int(-1)
                    rules.score_form(BF16, heads, rows, n, d, ctypes.byref(got))
                    assert got.value in (1, 2, 4)
                    assert got.value == 1 or got.value * 2 * 64 * d * 2 + (rows + 63) // 64 * 64 * 4 <= 160 * 1024


# heads, scores, kept rows of 256 bytes: the step in one launch took 0.71 to 0.79 times as long with the ranges of a head on all XCDs, or
# as long and more
@pytest.mark.parametrize("spread,sizes", [(1, [(5, 9000, 4000), (7, 9000, 4000), (9, 9000, 4000), (13, 9000, 4000)]),
                                          (0, [(3, 9000, 4000), (20, 9000, 4000), (1, 14000, 13000), (5, 2000, 1000), (32, 4096, 2048)])])
def test_ranges_on_all_xcds_where_that_is_faster(rules, spread, sizes):
    for heads, n, kept in sizes:
        assert rules.spreads_ranges(heads, rules.select_compact_parts(heads, n, kept, 256)) == spread, (heads, n, kept)


# heads, rows, keys, head_dim: row blocks of a workgroup with which the attention without key splits is fastest; the others took 1.08 to
# 2.2 times as long (heads that are no multiple of 8, of which an XCD has one more; rows of 32 elements in more than one round)
@pytest.mark.parametrize("blocks,sizes", [
    (2, [(36, 200, 555, 128), (36, 224, 1505, 128), (19, 350, 1536, 128), (9, 896, 335, 128), (11, 700, 1131, 128), (10, 700, 584, 96),
         (2, 1792, 5438, 128)]),
    (4, [(386, 112, 6144, 32), (217, 200, 4150, 32), (205, 256, 1441, 32), (301, 512, 6985, 32)]),
    (1, [(1, 100, 11889, 32), (28, 256, 9088, 32), (1, 64, 2743, 64)])])
def test_row_blocks_of_the_attention(rules, blocks, sizes):
    for size in sizes:
        assert rules.attention_row_waves(*size) == blocks, size


# more take longer for every size that was timed in 33 to 64
def test_at_most_32_key_splits(rules):
    for size in [(1, 64, 2743, 64), (2, 50, 2866, 128), (5, 32, 6383, 64), (1, 100, 11889, 32), (2, 64, 16446, 128), (1, 16, 1 << 20, 128)]:
        assert attention_shape(rules, *size, causal=0)[3] <= 32, size


# heads, kept rows, bytes of a row: whole steps took 0.5 to 0.98 times as long with ranges, or 1.01 times and more
@pytest.mark.parametrize("ranges,sizes", [
    (True, [(2, 11000, 256), (8, 30000, 256), (16, 13000, 256), (32, 8000, 128), (48, 3000, 192), (896, 2048, 256), (896, 7000, 256),
            (256, 13000, 256), (448, 2500, 512), (448, 300, 256), (112, 7000, 256), (896, 4000, 16)]),
    (False, [(448, 128, 256), (112, 2000, 192), (112, 19000, 32), (96, 10000, 16), (224, 3000, 80), (64, 128, 256), (8, 70000, 256)])])
def test_rows_in_ranges_where_it_is_faster(rules, ranges, sizes):
    for size in sizes:
        assert (rules.compact_parts(*size) > 0) == ranges, size


# heads, kept rows, bytes of a row, most rows of a head: uniform steps (0) of more than 16384 rows and ragged ones with few rows to move took
# 0.83 to 0.95 times as long with ranges, or 1.05 to 1.13 times
@pytest.mark.parametrize("ranges,sizes", [
    (True, [(24, 2613, 64, 0), (13, 1513, 160, 0), (2, 2322, 64, 0), (6, 906, 192, 0), (48, 1054, 256, 0), (8, 737, 192, 0),
            (40, 1880, 128, 1880), (12, 1170, 192, 1170), (28, 1338, 192, 1338), (56, 1084, 256, 1084), (38, 1023, 192, 1023), (24, 2074, 128, 3765),
            (46, 554, 256, 554), (2, 1514, 192, 3028), (36, 901, 256, 1867)]),
    (False, [(4, 509, 128, 0), (4, 152, 512, 0), (4, 244, 256, 0), (4, 427, 128, 0), (60, 129, 512, 129), (10, 242, 512, 242), (8, 563, 512, 563),
             (1, 1139, 512, 1139), (9, 869, 128, 869), (34, 266, 192, 532), (8, 715, 256, 920), (36, 274, 256, 711)])])
def test_few_rows_of_few_heads_in_ranges_where_it_is_faster(rules, ranges, sizes):
    for heads, kept, row, most in sizes:
        parts = rules.compact_ranges(heads, kept, most, row, ctypes.byref(ctypes.c_int(0))) if most else rules.compact_parts(heads, kept, row)
        assert (parts > 0) == ranges, (heads, kept, row, most)


# heads, kept rows, bytes of a row: epicache_compact took 0.8 to 0.97 times as long with ranges and a launch for their claims, or 1.02
# times and more
@pytest.mark.parametrize("ranges,sizes", [
    (True, [(1, 8192, 256), (2, 4096, 256), (4, 4096, 512), (4, 6144, 64), (8, 3072, 256), (16, 2048, 256), (32, 2048, 256), (63, 1024, 512),
            (896, 2048, 256), (640, 1500, 256), (120, 2526, 512), (112, 7000, 256), (896, 342, 256)]),
    (False, [(1, 3072, 256), (2, 2048, 256), (4, 3072, 128), (4, 2048, 512), (8, 2048, 256), (16, 1536, 256), (16, 1024, 512),
             (32, 1024, 512), (32, 1536, 256), (372, 1145, 256), (256, 1100, 256), (768, 700, 256)])])
def test_compact_with_a_workspace_takes_ranges_where_that_is_faster(rules, ranges, sizes):
    for size in sizes:
        taken = rules.compact_parts(*size) > 0 and bool(rules.compact_parts_pay_for_claims(*size))
        assert taken == ranges, size


def test_ranges_of_rows_fit_a_workgroup(rules):
    for heads in (1, 2, 8, 63, 64, 223, 224, 900, 65535):
        for kept in (1, 257, 4096, 4097, 16384, 32768, 40000):
            for row in (16, 48, 192, 256, 512, 1024):
                parts = rules.compact_parts(heads, kept, row)
                assert 0 <= parts <= 32
                if parts:
                    assert -(-kept // parts) <= 16 * (1024 // (row // 16))


def test_ranges_of_a_ragged_batch_hold_the_longest_head(rules):
    rows = ctypes.c_int(0)
    for heads in (1, 7, 64, 128, 225, 900, 65535):
        for kept in (300, 1025, 4096, 9000):
            for most in (kept, kept + 1, 3 * kept, 8 * kept):
                for row in (16, 48, 192, 256, 1024):
                    parts = rules.compact_ranges(heads, kept, most, row, ctypes.byref(rows))
                    assert 0 <= parts <= 32
                    if parts:
                        assert (parts - 1) * rows.value < most <= parts * rows.value, (heads, kept, most, row)
                        assert rows.value <= 16 * (1024 // (row // 16))
