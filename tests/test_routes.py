"""Which kernel, tile or order of tiles a size takes: the sizes at which the alternatives were measured, on the host alone
(the rules are functions of the library; no GPU is touched). A line that moves shows up here with the case that it moves."""
import ctypes
import os

import pytest

from oracle import ref
from paper_2411_09909_amd import binding


def rule(symbol, result, *arguments):
    """A function of the library's C++ side by its mangled name."""
    if not os.path.exists(binding.LIB_PATH):
        from paper_2411_09909_amd import build
        build.build(verbose=False)
    f = getattr(ctypes.CDLL(binding.LIB_PATH), symbol)
    f.restype, f.argtypes = result, arguments
    return f


E5, E4, FLOOR, ROUND = ref.FP8_E5M2, ref.FP8_E4M3, ref.E8M0_FLOOR, ref.E8M0_ROUND
i64, i32, f64, flag = ctypes.c_int64, ctypes.c_int, ctypes.c_double, ctypes.c_bool


def tile_order(tiles_m, tiles_n, tile_rows=256, tile_cols=256, batch=1):
    """(workgroups along x, rows of supertiles or 0 for equal runs)"""
    super_m = i32(-1)
    grid = rule("_ZN3amx14supertile_gridEiiiilRi", ctypes.c_uint, i32, i32, i32, i32, i64, ctypes.POINTER(i32))
    return grid(tiles_m, tiles_n, tile_rows, tile_cols, batch, ctypes.byref(super_m)), super_m.value


@pytest.mark.parametrize("tiles_m,tiles_n,tile_cols,runs", [
    (12, 20, 256, 1), (9, 112, 256, 1),   # fewer rounds (520 / 292 us, 556 / 392)
    (8, 16, 256, 1), (1, 126, 256, 1), (9, 16, 256, 1), (12, 16, 128, 0),  # one round: 98 / 76, 193 / 123, 87 / 77, 28 / 29
    (2, 112, 256, 1), (3, 172, 128, 1), (8, 40, 256, 1), (14, 20, 256, 1), (6, 112, 256, 1),
    (6, 86, 128, 0), (4, 224, 128, 0), (10, 32, 256, 0), (12, 43, 256, 0), (14, 43, 256, 0), (3, 86, 256, 0),
    (32, 2, 256, 0), (16, 112, 256, 0), (8, 32, 256, 0)])
def test_order_of_tiles_that_fill_a_compute_unit(tiles_m, tiles_n, tile_cols, runs):
    grid, super_m = tile_order(tiles_m, tiles_n, 256, tile_cols)
    assert (super_m == 0) == bool(runs)


@pytest.mark.parametrize("tiles_m,tiles_n,rows,batch,runs", [(4, 4, 256, 8, 1), (24, 4, 64, 1, 1), (10, 32, 256, 4, 1),
                                                             (8, 32, 256, 4, 0)])
def test_order_in_a_batch_and_of_small_tiles(tiles_m, tiles_n, rows, batch, runs):
    """Runs wherever a fifth of the slots is empty."""
    assert (tile_order(tiles_m, tiles_n, rows, 256, batch)[1] == 0) == bool(runs)


@pytest.mark.parametrize("group,rows,groups,batch,log2", [
    (32, 4096, 256, 1, 3), (16, 4096, 512, 1, 3), (64, 4096, 128, 1, 2), (128, 4096, 64, 1, 1), (32, 128, 126, 32, 3),
    (32, 32, 32, 1, 0), (32, 4096, 16, 1, 2), (32, 128, 48, 8, 2),                                     # few workgroups
    (32, 1000000, 1, 1, 0), (32, 128, 1, 4096, 0), (32, 1000000, 2, 1, 1), (16, 1000000, 3, 1, 2),     # 29.1 / 15.3, 16.0 / 8.9
    (32, 65536, 5, 1, 3), (128, 1000000, 1, 1, 0), (64, 1000000, 1, 1, 0), (64, 1000000, 2, 1, 1)])
def test_groups_to_a_workgroup_of_the_strided_cast(group, rows, groups, batch, log2):
    """No more waves than there are groups (us with eight to a workgroup / as many as there are)."""
    assert rule("_ZN3amx18strided_waves_log2Eilll", i32, i32, i64, i64, i64)(group, rows, groups, batch) == log2


@pytest.mark.parametrize("groups_log2,rows,groups,batch,lines,log2", [
    (0, 12086, 1, 32, 0, 2), (0, 752, 1, 512, 0, 2), (0, 128, 2, 1, 1, 1), (0, 64, 1, 512, 1, 0), (0, 334, 1, 1, 0, 2),  # 9.5 / 5.9 us, 8.4 / 5.2
    (0, 2300, 8, 1, 0, 1), (0, 1782, 8, 1, 0, 0), (0, 128, 190, 1, 1, 0), (1, 8163, 2, 64, 0, 1), (1, 130, 2, 300, 0, 1),
    (1, 128, 2, 300, 1, 0), (1, 128, 2, 512, 1, 1), (3, 4096, 256, 1, 1, 0)])
def test_rows_to_a_workgroup_of_the_strided_cast(groups_log2, rows, groups, batch, lines, log2):
    """Four waves to a workgroup where the groups are fewer, unless that leaves compute units idle (one wave / four)."""
    rows_log2 = rule("_ZN3amx17strided_rows_log2Eilllb", i32, i32, i64, i64, i64, flag)
    assert rows_log2(groups_log2, rows, groups, batch, bool(lines)) == log2


@pytest.mark.parametrize("rows,groups,batch,one", [
    (18, 12, 64, 1), (64, 3, 512, 1), (65, 12, 64, 0), (128, 32, 32, 0), (129, 24, 32, 1), (256, 3, 512, 1),  # 8.3 / 5.7 us; 7.1 / 8.6; 15.8 / 13.8
    (257, 3, 70, 1), (257, 3, 77, 0), (8964, 7, 1, 1), (14169, 28, 1, 0)])                                    # 10.6 / 8.3; 35 / 38
def test_wide_groups_of_the_strided_cast(rows, groups, batch, one):
    """Steps along K that are no whole lines, groups of 128: two of them to a workgroup / one, of up to 256 rows."""
    assert rule("_ZN3amx22strided_one_wide_groupElll", flag, i64, i64, i64)(rows, groups, batch) == bool(one)


@pytest.mark.parametrize("Hq,Hkv,Sq,D,tiles,splits,here", [
    (32, 8, 1, 128, 1, 4, 0), (8192, 1024, 1, 64, 1, 1, 0), (128, 16, 2, 128, 1, 64, 0),                  # one tile: 15.7 / 9.8 us, but 13.3 / 15.8
    (32, 8, 1, 64, 2, 63, 1), (32, 8, 1, 64, 2, 64, 0), (4096, 1024, 1, 64, 2, 16, 0), (32, 8, 1, 128, 2, 64, 1),   # two: 56.8 / 46.1
    (816, 408, 1, 64, 3, 78, 0), (64, 8, 1, 64, 3, 2048, 1), (816, 408, 1, 64, 3, 40, 1), (816, 408, 1, 64, 4, 78, 1),  # three: 122 / 110
    (816, 408, 1, 128, 3, 78, 1), (34, 2, 1, 128, 8, 64, 0)])
def test_decode_attention_of_short_ranges(Hq, Hkv, Sq, D, tiles, splits, here):
    """The kernel of 16 columns and four waves to a range / the other one."""
    f = rule("_ZN3amx29attention_decode_16_preferredEllllii", flag, i64, i64, i64, i64, i32, i32)
    assert f(Hq, Hkv, Sq, D, tiles, splits) == bool(here)


ROWS, ROWS_CACHED, COLUMNS = 0, 1, 2


@pytest.mark.parametrize("M,ldc,K,way,base", [
    (2048, 11008, 4096, ROWS, 0), (1504, 4096, 14336, ROWS, 0), (4096, 4096, 512, ROWS, 0),        # whole lines: 68.3 / 67.2 row by row
    (2048, 8192, 512, COLUMNS, 0), (4096, 16384, 1024, COLUMNS, 0), (64, 32768, 128, COLUMNS, 64),  # 24.0 / 30.1; half lines 53 / 66
    (2048, 24576, 512, ROWS, 0), (2048, 8192, 1024, ROWS_CACHED, 4), (4096, 8208, 1024, ROWS, 0),   # 55.2 / 50.6; 119 / 86
    (3000, 5001, 4096, ROWS_CACHED, 0), (4096, 32001, 4096, ROWS, 0), (4096, 4545, 4544, ROWS, 0)])
def test_order_and_policy_of_the_stores(M, ldc, K, way, base):
    """us column by column / row by row (rows that are not even half lines: through the caches below 80 MB of C and up to K 4096)"""
    store_way = rule("_ZN3amx9store_wayEPKflll", i32, ctypes.c_void_p, i64, i64, i64)
    assert store_way(1 << 20 | base, M, K, 4 * ldc) == way


def test_grid_has_a_workgroup_for_every_tile():
    for tiles_m in range(1, 40):
        for tiles_n in range(1, 70):
            for batch in (1, 2):
                grid, super_m = tile_order(tiles_m, tiles_n, batch=batch)
                assert grid % 8 == 0 and grid >= tiles_m * tiles_n
                if super_m:
                    assert super_m == -(-tiles_m // 8) and grid == 8 * 32 * -(-(super_m * -(-tiles_n // 4)) // 8)
                else:
                    assert grid < tiles_m * tiles_n + 8


@pytest.mark.parametrize("M,N,tile", [
    (2048, 11008, 2), (1900, 10240, 2), (2600, 8192, 2), (3800, 4544, 2),  # 257 .. 384 large tiles (213 / 183, 403 / 339, ...)
    (768, 22016, 2), (768, 28672, 1), (640, 32001, 1),                     # three rows of them: 258, 336, 378 large tiles
    (256, 11008, 3), (500, 4096, 3), (4096, 28672, 1), (4096, 4096, 1)])
def test_tile_of_the_bf16_panel_kernel(M, N, tile):
    """1: 256 x 256, 2: 256 x 128, 3: 64 x 256"""
    assert rule("_ZN3amx16bf16_tile_choiceElll", i32, i64, i64, i64)(M, N, 1) == tile


@pytest.mark.parametrize("M,N,K,fp4", [
    (2048, 4096, 128, 1), (512, 4096, 4096, 0), (1024, 4096, 2048, 0),         # 20 / 12.6 us, 19 / 31.6, 20 / 23
    (32768, 128, 128, 1), (100000, 512, 128, 1),                               # 12.2 / 10.3, 104 / 47
    (80, 28672, 8192, 1), (256, 28672, 8192, 1), (64, 28672, 8192, 0), (96, 4096, 4096, 0), (4096, 4096, 4096, 1)])
def test_symmetric_power_of_two_scales_of_many_rows(M, N, K, fp4):
    """The FP4 kernel or the one that reads both operands as packed codes, in one launch."""
    assert rule("_ZN3amx16fp4_beats_streamEllld", flag, i64, i64, i64, f64)(M, N, K, 4.0) == bool(fp4)


def one_launch(scale, asym, M, N, K, batch=1, group=32, scaled=False):
    """Whether the product goes to the kernel that reads both operands as packed codes."""
    f = rule("_ZN3amx21stream_path_preferredEiblbllll", flag, i32, flag, i64, flag, i64, i64, i64, i64)
    return f(scale, bool(asym), group, scaled, M, N, K, batch)


def one_launch_gated(scale, asym, M, N, K, group=32):
    return rule("_ZN3amx20stream_glu_preferredEibllll", flag, i32, flag, i64, i64, i64, i64)(scale, bool(asym), group, M, N, K)


@pytest.mark.parametrize("scale,asym,M,N,K,here", [
    (E5, 1, 1, 4096, 4096, 1), (E5, 1, 64, 28672, 8192, 1), (E5, 0, 64, 11008, 4096, 1),
    (E5, 1, 32, 1024, 28672, 0), (E5, 1, 32, 1024, 16384, 1), (E5, 1, 32, 4096, 28672, 0),  # 27 / 22 us, 16.6 / 17.5, 27.4 / 25.2
    (E5, 1, 64, 128, 24576, 0), (E5, 1, 64, 8192, 28672, 0), (E5, 1, 1, 512, 40960, 0), (E5, 1, 1, 512, 28672, 1),
    (E5, 1, 32, 32, 16384, 0), (E5, 0, 32, 512, 65536, 0), (E5, 0, 17, 512, 40960, 1), (E5, 0, 1, 512, 65536, 1),
    (E4, 1, 32, 1024, 16384, 1), (E4, 1, 32, 1024, 28672, 0)])
def test_few_rows_and_a_long_k(scale, asym, M, N, K, here):
    """Up to 64 rows: one launch, unless K is so long that the few-rows kernel's slices of it are faster."""
    assert one_launch(scale, asym, M, N, K) == bool(here)
    assert one_launch(scale, asym, M, N, K, scaled=True) and one_launch(scale, asym, M, N, K, group=16)
    assert one_launch_gated(scale, asym, M, N, K)


@pytest.mark.parametrize("asym,batch,M,N,K,here", [
    (1, 32, 64, 4096, 1024, 0), (1, 512, 64, 512, 256, 0), (1, 64, 48, 2048, 512, 0), (0, 64, 48, 2048, 512, 0),
    (1, 32, 64, 2048, 1024, 1), (1, 512, 64, 128, 4096, 1), (0, 24, 48, 2048, 512, 1), (1, 24, 48, 2048, 512, 1),
    (1, 32, 32, 4096, 1024, 1),
    (1, 512, 16, 512, 256, 1), (1, 2, 64, 4096, 1024, 1)])
def test_batches_of_few_rows(asym, batch, M, N, K, here):
    """Two rounds of workgroups and 33 to 64 rows each: the few-rows kernel, which dequantizes A once, for a short K or many
    columns (38.4 / 34.5 us, 51 / 33, 29.6 / 24.3, 24.2 / 22.6; but 21 / 23, 66 / 170, 11.9 / 13.8, 14.5 / 14.7)."""
    assert one_launch(E5, asym, M, N, K, batch) == bool(here)


@pytest.mark.parametrize("asym", [0, 1])
@pytest.mark.parametrize("M,N,K", [(40, 4096, 288), (300, 4096, 4096), (800, 4096, 512)])
def test_rounded_power_of_two_scales_stay_where_their_largest_values_are_finite(M, N, K, asym):
    assert not one_launch(ROUND, asym, M, N, K) and not one_launch_gated(ROUND, asym, M, N, K)


@pytest.mark.parametrize("scale,asym,M,N,K,here", [
    (E5, 1, 256, 4096, 4096, 1), (E5, 1, 256, 11008, 4096, 1), (E5, 1, 96, 10240, 8192, 0), (E5, 1, 256, 5120, 13824, 0),
    (E5, 1, 256, 32001, 4096, 0), (E5, 0, 256, 32001, 4096, 1), (E5, 1, 256, 28672, 8192, 0),
    (E5, 1, 512, 4096, 4096, 1), (E5, 1, 512, 4096, 11008, 1), (E5, 1, 448, 11008, 4096, 1), (E5, 1, 512, 11008, 4096, 0),
    (E5, 1, 640, 8192, 8192, 1), (E5, 1, 768, 8192, 8192, 0), (E5, 1, 448, 4544, 4544, 1), (E5, 1, 512, 4544, 4544, 0),
    (E5, 1, 768, 1024, 1024, 1), (E5, 1, 769, 1024, 1024, 0), (FLOOR, 1, 256, 4096, 4096, 1), (FLOOR, 1, 257, 4096, 4096, 0)])
def test_routes_of_65_to_768_rows(scale, asym, M, N, K, here):
    """us, this kernel / the other: 17 / 50, 40 / 79, 45 / 35, 74 / 70, 99 / 83, 73 / 78, 177 / 151; 27 / 44, 63 / 106, 62 / 65,
    73 / 66, 110 / 116, 133 / 121, 43 / 50, 58 / 51; the ends of the range"""
    assert one_launch(scale, asym, M, N, K) == bool(here)


@pytest.mark.parametrize("scale,asym,group,scaled,M,N,K,here", [
    (E5, 0, 32, 0, 768, 8192, 8192, 1), (E5, 0, 32, 0, 769, 8192, 8192, 0),           # 149 / 99; prepared weights alone
    (E5, 0, 32, 0, 700, 4096, 14336, 1), (E5, 1, 32, 0, 700, 4096, 14336, 1),
    (E4, 0, 16, 1, 320, 8192, 28672, 1), (E4, 0, 16, 1, 640, 28672, 8192, 1),         # 466 / 167, 461 / 311
    (E4, 0, 16, 1, 1500, 28672, 8192, 0), (E4, 0, 16, 1, 1343, 6144, 4096, 0),        # 645 / 770, 71 / 81
    (E4, 0, 16, 1, 550, 13952, 512, 0), (E5, 0, 32, 0, 547, 8960, 3072, 0),           # 20 / 26; prepared 32 / 36
    (E5, 0, 32, 0, 400, 28672, 8192, 0), (E5, 0, 32, 0, 160, 28672, 8192, 1), (E5, 0, 32, 0, 90, 8960, 28672, 0),  # 110 / 102, 72 / 94
    (E4, 0, 16, 1, 1500, 1024, 14336, 1), (E4, 0, 16, 1, 1501, 1024, 14336, 0)])
def test_routes_of_weights_that_come_from_memory(scale, asym, group, scaled, M, N, K, here):
    """us on the panels / on this kernel, three sets of buffers in turn."""
    assert one_launch(scale, asym, M, N, K, 1, group, bool(scaled)) == bool(here)


@pytest.mark.parametrize("scale,asym,group,scaled,M,N,K,here", [
    (E5, 0, 32, 0, 548, 11008, 4096, 0), (E5, 0, 32, 0, 576, 11296, 6400, 0), (E5, 0, 32, 0, 525, 17792, 6144, 0),  # prepared 51 / 61, 71 / 94, 94 / 131
    (E4, 0, 16, 1, 1344, 4096, 14336, 0), (E4, 0, 16, 1, 973, 8192, 8192, 0), (E4, 0, 16, 1, 1138, 5120, 13824, 0),  # 161 / 171, 139 / 148, 167 / 178
    (E5, 0, 32, 0, 548, 4096, 4096, 1), (E5, 0, 32, 0, 700, 8192, 8192, 1), (E4, 0, 16, 1, 901, 4096, 4096, 1), (E4, 0, 16, 1, 1200, 1024, 14336, 1)])
def test_routes_of_weights_that_stay_in_the_caches(scale, asym, group, scaled, M, N, K, here):
    """us on the panels / on this kernel, the same buffers again and again."""
    assert one_launch(scale, asym, M, N, K, 1, group, bool(scaled)) == bool(here)


@pytest.mark.parametrize("scale,asym,M,N,K,here", [(E5, 1, 256, 28672, 8192, 1), (E5, 1, 257, 28672, 8192, 0),
                                                   (FLOOR, 1, 256, 22016, 4096, 0), (FLOOR, 1, 128, 22016, 4096, 1),
                                                   (FLOOR, 0, 800, 11008, 1024, 0)])
def test_routes_of_the_gated_product(scale, asym, M, N, K, here):
    """Up to 256 rows its other kernel is a tiled one: large weights stay (177 / 350)."""
    assert one_launch_gated(scale, asym, M, N, K) == bool(here)


@pytest.mark.parametrize("scale,group", [(E5, 32), (E4, 32), (E4, 16), (FLOOR, 32), (FLOOR, 16), (ROUND, 32)])
def test_beyond_256_rows_the_gated_product_goes_where_the_plain_one_does(scale, group):
    """Their sums are promised to be the same bits there (but for products that the few-rows kernel takes against large weights)."""
    for asym in (0, 1):
        for M in (257, 300, 384, 448, 512, 513, 640, 768, 769, 1504, 4096, 20000):
            for N in (64, 1024, 2048, 5632, 11008, 22016, 28672):
                for K in (96, 256, 1024, 2048, 4096, 8192, 11008):
                    assert one_launch_gated(scale, asym, M, N, K, group) == one_launch(scale, asym, M, N, K, 1, group)


@pytest.mark.parametrize("workgroups,Sq,Sk,causal,pairs", [
    (672, 2688, 2688, 1, 1), (768, 3072, 3072, 1, 0),                        # 93 / 88 us, 114 / 119
    (512, 2048, 2048, 0, 1), (600, 1920, 1920, 0, 0), (704, 1344, 1344, 0, 0),  # without a mask: 101 / 118, 77 / 89
    (640, 2560, 2720, 1, 1), (640, 2560, 3840, 1, 0), (500, 2000, 4000, 1, 1),  # more keys than queries
    (64, 96, 96, 1, 0), (64, 288, 288, 0, 0), (64, 352, 352, 1, 1), (64, 128, 128, 1, 1)])  # odd numbers of key tiles
def test_attention_walks_over_pairs_of_key_tiles(workgroups, Sq, Sk, causal, pairs):
    """Tile by tile / pairs: workgroups of the same length must all run at once, two to a compute unit."""
    assert rule("_ZN3amx9pairs_payEllli", flag, i64, i64, i64, i32)(workgroups, Sq, Sk, causal) == bool(pairs)


@pytest.mark.parametrize("M,N,K,gated,prepared,tile", [
    (1504, 6144, 4096, 0, 0, 7), (1563, 10240, 8192, 0, 0, 4), (1504, 4096, 14336, 0, 0, 5), (2048, 11008, 4096, 0, 0, 4),
    (281, 8192, 8192, 0, 0, 6),
    (2071, 13824, 5120, 1, 0, 1), (1148, 25920, 2432, 1, 1, 1),  # 192 x 256 would take a third round (260 / 281, 120 / 140 us)
    (1311, 11072, 1792, 1, 0, 3), (574, 24704, 1792, 0, 0, 3),   # or a second one, with a short K (65 / 72, 82 / 87)
    (1312, 11264, 2048, 1, 0, 3), (1408, 5632, 1024, 1, 0, 3),   # 276 / 280 (the layer), 25.1 / 25.7
    (768, 22016, 4096, 1, 0, 2), (768, 22016, 4096, 0, 0, 4),    # gated 189 / 196
    (803, 8192, 8192, 0, 1, 2), (696, 10240, 8192, 0, 1, 2), (1577, 4096, 11008, 0, 1, 2),  # prepared: 124 / 136, 126 / 138, 159 / 162
    (836, 8192, 28672, 0, 0, 2), (2029, 4096, 4096, 0, 0, 2), (1600, 4096, 4096, 0, 0, 2),  # 571 / 584, 64 / 66, 56.5 / 57.2
    (1805, 4096, 14336, 0, 0, 7), (1611, 4096, 11008, 0, 0, 7), (1493, 4544, 4544, 0, 0, 7)])  # ratios 0.88, 0.94, 0.98
def test_tile_that_the_bf16_panel_kernel_runs(M, N, K, gated, prepared, tile):
    """1: 256 x 256, 2: 256 x 128, 3: 64 x 256, 4: 192 x 256, 5: 192 x 128, 6: 128 x 128, 7: 192 x 192. The sizes behind each
    line; in brackets what the shape that stays / the other one takes."""
    bf16_tile = rule("_ZN3amx9bf16_tileEllllbbb", i32, i64, i64, i64, i64, flag, flag, flag)
    assert bf16_tile(M, N, K, 1, bool(gated), bool(prepared), True) == tile


@pytest.mark.parametrize("M,N,K,whole,ragged", [
    (1323, 11008, 4096, 4, 3), (2570, 6144, 4096, 4, 3), (1124, 13824, 5120, 4, 4),  # 167 / 183 us, 170 / 177, ratio 0.93
    (1349, 16384, 2048, 4, 2), (1498, 11008, 4096, 4, 4)])                           # 144 / 149, 0.94 to 1.02
def test_tile_where_rows_of_c_are_no_whole_lines(M, N, K, whole, ragged):
    bf16_tile = rule("_ZN3amx9bf16_tileEllllbbb", i32, i64, i64, i64, i64, flag, flag, flag)
    assert [bf16_tile(M, N, K, 1, False, False, w) for w in (True, False)] == [whole, ragged]


@pytest.mark.parametrize("M,N,K,lines,cut", [
    (4096, 28672, 8192, 1, 8192), (1192, 28672, 8192, 1, 13056), (1504, 28672, 4096, 1, 10752),
    (3000, 10240, 8192, 1, 0),                              # 160 MB: 406 / 413 us
    (2546, 22016, 4096, 1, 0), (1563, 22016, 4096, 1, 0),   # 172 MB, more than five rows of tiles: 388 / 408, gated 286 / 300
    (2400, 26624, 4096, 1, 0), (2900, 27648, 5120, 1, 0),   # a last round of hardly any tiles: ratios 1.07, 1.02
    (2400, 28672, 4096, 0, 0), (1504, 28672, 4096, 0, 0),   # rows of C that are no whole lines: 613 / 642, 426 / 437
    (973, 32001, 4096, 0, 0), (2048, 28672, 8192, 0, 8192)])  # 341 / 353, 976 / 931
def test_columns_whose_weights_are_expanded_at_a_time(M, N, K, lines, cut):
    """Whole / in pieces (0: whole) on tiles of 256 x 256."""
    at_a_time = rule("_ZN3amx22bf16_columns_at_a_timeEillllb", i64, i32, i64, i64, i64, i64, flag)(1, M, N, K, 1, bool(lines))
    assert at_a_time == (cut or N)
