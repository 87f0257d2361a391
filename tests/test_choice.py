"""Which way the library runs a call, by its own choice (a host function: no GPU)."""
import os

import pytest

torch = pytest.importorskip("torch")
LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_13313_amd", "libozimmu.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libozimmu.so not built")


@pytest.fixture(scope="module")
def oz():
    from paper_2409_13313_amd import ozimmu
    return ozimmu


@pytest.mark.parametrize("m,n,p", [(47, 11948, 48), (1, 4096, 1), (64, 20001, 97), (300, 5937, 174)])
@pytest.mark.parametrize("k", range(3, 17))
def test_one_scale_per_slice_is_never_cut_whatever_the_room(oz, m, n, p, k):
    # (the sums of cut tiles are added up with one exponent per row and column)
    assert oz.choose(m, n, p, k, "per_slice", "per_pair", workspace_bytes=1 << 34).parts == 1
    assert oz.choose(m, n, p, 3, "rn", "grouped", workspace_bytes=1 << 34).parts > 1


# (measured with rows of D that begin inside a memory line, kept in L2 and streamed past it, us)
@pytest.mark.parametrize("m,n,p,k,accumulate,kept,streamed", [
    (1011, 34, 20402, 3, "grouped", 55.6, 131.9), (3440, 31, 6195, 5, "grouped", 65.7, 129.8), (554, 5, 20266, 10, "grouped", 94.9, 104.5),
    (249, 3, 117287, 9, "grouped", 261.8, 300.7), (374, 114, 84687, 4, "per_pair", 167.5, 209.5), (169, 1, 120809, 6, "grouped", 120.7, 153.9),
    (97567, 95, 106, 7, "grouped", 158.4, 147.8), (68693, 119, 285, 8, "grouped", 191.3, 183.0), (280, 3, 77204, 12, "grouped", 195.2, 184.6),
    (88, 24, 135175, 9, "grouped", 154.8, 147.6), (133562, 2, 213, 6, "per_pair", 303.1, 291.8), (129710, 145, 65, 3, "per_pair", 138.4, 129.4)])
def test_rows_are_kept_in_the_cache_where_that_is_faster(oz, m, n, p, k, accumulate, kept, streamed):
    assert oz.choose(m, n, p, k, "rn", accumulate).merge_rows == (kept < streamed)


# (measured with 32 x 32 tiles, two to a compute unit, and with the tile that was the next best, us)
@pytest.mark.parametrize("m,n,p,k,accumulate,small,other", [
    (9998, 67, 320, 14, "grouped", 61.0, 73.9), (5000, 200, 500, 14, "grouped", 62.2, 74.8), (7552, 80, 393, 11, "grouped", 45.4, 48.0),
    (70484, 1, 109, 6, "per_pair", 118.7, 128.0), (1500, 1000, 1500, 12, "grouped", 127.7, 124.2),
    (216, 1, 105570, 12, "grouped", 225.1, 212.5), (1936, 53, 14344, 12, "grouped", 216.9, 195.7), (447, 31, 33552, 11, "grouped", 119.0, 114.1)])
def test_the_smallest_tiles_where_their_steps_cover_their_ends(oz, m, n, p, k, accumulate, small, other):
    choice = oz.choose(m, n, p, k, "rn", accumulate)
    assert oz.WAYS[choice.way] == "resident"
    assert (oz.resident_tile(n, k, accumulate, choice.tile) == (32, 32)) == (small < other)


# (measured whole and in the parts that were chosen, or are, us; the same split)
@pytest.mark.parametrize("m,n,p,k,accumulate,whole,cut", [
    (8, 2054, 8, 10, "per_pair", 31.2, 45.2), (2, 2465, 19, 8, "per_pair", 27.7, 35.2), (33, 3385, 232, 10, "per_pair", 44.6, 53.9),
    (103, 3720, 8, 9, "per_pair", 40.1, 45.2), (297, 4429, 88, 10, "per_pair", 56.4, 60.7), (21, 2761, 6, 6, "per_pair", 24.6, 27.4),
    (477, 4256, 8, 10, "per_pair", 54.7, 58.7), (9, 6694, 26, 3, "grouped", 35.4, 20.4)])
def test_tiles_are_cut_where_that_is_faster(oz, m, n, p, k, accumulate, whole, cut):
    assert (oz.choose(m, n, p, k, "rn", accumulate).parts > 1) == (cut < whole)


# (measured in one launch, or the launches of cut columns, and in two along the inner dimension, us, whole calls)
@pytest.mark.parametrize("m,n,p,k,whole,cut", [
    (12, 1982, 3483, 8, 47.7, 61.2), (8, 2369, 4391, 3, 55.2, 66.4), (5, 2756, 1415, 3, 31.6, 37.1), (58, 1583, 4548, 7, 60.6, 66.8),
    (14, 1992, 4768, 9, 69.6, 76.1), (1, 1306, 2569, 12, 43.6, 46.6), (31, 1624, 1920, 6, 26.0, 32.5),
    (47, 11948, 48, 8, 58.4, 31.4), (256, 8192, 256, 8, 63.6, 48.9), (12, 17700, 942, 14, 245.5, 212.0), (1, 13311, 545, 13, 112.8, 93.0), (27, 6332, 560, 3, 30.4, 25.7), (13, 10255, 295, 4, 48.9, 34.4),
    (142, 11505, 66, 8, 67.1, 39.5), (37, 2031, 130, 8, 21.7, 23.7), (22, 2240, 170, 13, 38.4, 35.4), (7, 2613, 2, 3, 15.3, 19.8), (500, 1024, 500, 8, 23.2, 26.1)])
def test_vectors_are_split_along_the_inner_dimension_where_that_is_faster(oz, m, n, p, k, whole, cut):
    assert (oz.SPLIT_WAYS[oz.choose(m, n, p, k).split_way] == "cut") == (cut < whole)


# (measured with k_held's tile and with the best of the others, us, whole calls)
@pytest.mark.parametrize("m,n,p,k,held,other", [
    (8532, 421, 5453, 8, 612.9, 531.7), (7595, 240, 357, 8, 43.8, 38.3), (1701, 159, 3116, 11, 80.3, 71.5), (1081, 70, 5947, 10, 67.0, 59.7),
    (1409, 65, 805, 13, 26.4, 22.9), (215, 203, 5345, 13, 40.2, 34.8), (780, 6178, 1346, 14, 579.3, 518.8), (2446, 6611, 444, 14, 646.4, 581.1),
    (2017, 193, 824, 11, 34.3, 39.5), (1387, 59, 1565, 9, 22.5, 26.4), (1621, 114, 4056, 9, 56.9, 64.9), (804, 386, 5432, 13, 130.8, 150.5),
    (2105, 2105, 2105, 13, 508.5, 581.1), (759, 8816, 1462, 11, 554.4, 653.0), (2788, 16786, 2762, 5, 1499.2, 1746.3), (2000, 600, 2000, 6, 52.6, 51.2), (1537, 2051, 1283, 9, 149.0, 157.3), (1424, 1424, 1424, 9, 107.7, 113.2), (6981, 1090, 895, 7, 160.5, 181.0),
    (4708, 5, 409, 10, 26.0, 24.0), (3136, 1631, 2097, 10, 436.8, 415.5), (2462, 7133, 2808, 6, 828.7, 795.7), (2541, 712, 2488, 10, 205.6, 197.6),
    (801, 2368, 10172, 7, 493.6, 480.8), (8192, 8192, 8192, 6, 6701.7, 7039.9), (8192, 8192, 8192, 8, 11580.0, 11420.0),
    (6144, 6144, 6144, 11, 8316.0, 8774.0), (6144, 6144, 6144, 8, 4761.0, 4897.0), (16384, 16384, 16384, 9, 114243.0, 111196.0)])
def test_slices_of_a_are_held_where_that_is_faster(oz, m, n, p, k, held, other):
    assert (oz.choose(m, n, p, k).tile == oz.HELD_TILE) == (held < other)


# (measured with whole columns, or the cut of many launches, and with columns cut along the inner dimension beside rows, us, whole calls)
@pytest.mark.parametrize("m,n,p,k,accumulate,whole,cut", [
    (11, 7698, 2231, 5, "grouped", 92.8, 117.5), (10, 5261, 2140, 4, "grouped", 58.1, 72.9), (704, 13298, 1524, 5, "grouped", 330.1, 361.3),
    (1045, 8580, 8, 4, "grouped", 45.1, 51.7), (8, 9356, 2100, 4, "per_pair", 99.1, 124.3), (754, 5777, 2091, 6, "per_pair", 219.0, 235.5),
    (352, 4636, 1844, 11, "grouped", 182.5, 192.1), (736, 9172, 1735, 7, "grouped", 313.8, 329.5), (701, 16385, 1513, 5, "grouped", 395.8, 421.7),
    (640, 14848, 256, 8, "grouped", 141.0, 128.8), (909, 14947, 85, 4, "grouped", 88.5, 72.3), (523, 31111, 815, 8, "grouped", 736.8, 672.6),
    (1024, 16384, 1024, 8, "grouped", 535.4, 505.2), (448, 57799, 128, 14, "wide", 643.7, 515.3), (33, 56249, 2084, 9, "grouped", 1141.5, 980.5),
    (1300, 8190, 901, 20, "grouped", 2001.4, 1971.4), (488, 7153, 1075, 17, "grouped", 652.8, 615.1), (44, 5720, 1762, 16, "grouped", 144.4, 164.0), (325, 7969, 1875, 6, "grouped", 171.4, 191.1),
    (28, 12427, 2068, 14, "grouped", 338.2, 292.4), (57, 156679, 812, 14, "grouped", 1863.8, 1582.4), (232, 56640, 1927, 9, "grouped", 1567.2, 1554.4)])
def test_columns_are_cut_beside_rows_where_that_is_faster(oz, m, n, p, k, accumulate, whole, cut):
    assert (oz.SPLIT_WAYS[oz.choose(m, n, p, k, "rn", accumulate).split_way] == "cut_columns") == (cut < whole)


def test_two_operands_of_columns_are_cut_beside_each_other(oz):
    # (what the GPU test of that kernel calls, in its workspace; with A by rows and B transposed there is nothing to cut)
    m, n, p, k = 256, 40001, 700, 8
    room = oz.workspace_bytes(m, n, p, k) + (64 << 20)
    assert oz.split_way(True, False, m, n, p, k, room) == "cut_columns" and oz.split_way(False, True, m, n, p, k, room) != "cut_columns"
