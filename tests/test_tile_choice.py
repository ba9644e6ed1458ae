"""Host-side choices behind the products and contractions (csrc/tile_choice.hpp), compiled as plain C++."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "tile_choice.hpp"
using namespace givens;
extern "C" {
unsigned order(unsigned block, unsigned total) { return xcd_order(block, total); }
int product(int m, int k, long long B, int units, int cplx) { return product_tile(m, k, B, units, cplx != 0); }
double contraction_us(int tile, int slices, int rows, long long B, int units)
{
    const TileCost &t = kGramCost[0][tile];
    const long long tiles = (long long)((rows + t.bm - 1) / t.bm) * ((rows + t.bn - 1) / t.bn);
    return tile_time(t, (tiles * slices + 7) / 8, ((B + slices - 1) / slices + kGramK - 1) / kGramK, units);
}
void plan(int rows, long long B, int units, int cplx, int *slices, long long *cols)
{
    const GramPlan p = gram_plan(rows, B, units, cplx != 0);
    *slices = p.slices;
    *cols = p.cols;
}
int listed(int P, int units, long long runs, long long per, int active) { return tile_apply_listed(P, units, runs, per, active); }
int pairs_listed(int P, int units) { return tile_pairs_listed(P, units); }
}
"""


@pytest.fixture(scope="module")
def choice(tmp_path_factory):
    folder = tmp_path_factory.mktemp("tile_choice")
    source, library = str(folder / "choice.cpp"), str(folder / "libchoice.so")
    with open(source, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-I" + os.path.join(ROOT, "paper_2106_00003_amd", "csrc"), source, "-o", library], check=True)
    lib = ctypes.CDLL(library)
    lib.contraction_us.restype = ctypes.c_double
    return lib


# A contraction's workgroups reach the eight XCDs in turn; whatever their number, each XCD has consecutive ones of the list.
# n = 314, B = 15395 in 60 slices of 25 tiles: 70 us with the list handed out in turn, 38 so.
def test_every_xcd_has_a_consecutive_part_of_the_list(choice):
    for total in [*range(1, 130), 1500, 1504, 1530]:
        places = [choice.order(b, total) for b in range(total)]
        assert sorted(places) == list(range(total))
        for xcd in range(8):
            part = places[xcd::8]
            assert part == list(range(part[0], part[0] + len(part))) if part else total < 8


# Times of products measured with every tile (64 x 64, 128 x 64, 128 x 128, 256 x 128), in us: the choice is one of the fastest.
# Many have a few workgroups more than there are compute units, which takes as long as one more on every unit.
@pytest.mark.parametrize("cplx,n,B,us", [
    (False, 1024, 4525, (81.4, 85.8, 88.8, 98.9)), (False, 640, 6784, (50.9, 54.9, 57.6, 65.1)),
    (False, 512, 9856, (44.5, 48.2, 50.9, 54.7)), (False, 512, 10176, (45.0, 48.3, 51.2, 55.3)),
    (False, 314, 15395, (28.6, 30.7, 33.0, 37.6)), (False, 162, 24440, (19.6, 21.2, 24.3, 25.4)),
    (False, 256, 16819, (24.2, 27.2, 27.9, 30.9)), (False, 566, 43171, (205.8, 202.1, 182.0, 216.8)),
    (False, 896, 3491, (51.6, 45.1, 53.7, 86.9)), (False, 896, 3048, (43.8, 47.4, 54.9, 87.4)),
    (False, 64, 4417, (4.2, 5.2, 7.8, 11.5)), (False, 1000, 3200, (56.5, 50.5, 60.1, 96.7)),
    (False, 1316, 4919, (145.5, 134.2, 117.0, 130.0)), (False, 2048, 7218, (444.5, 387.4, 352.1, 294.8)),
    (False, 1000, 27456, (392.9, 345.9, 317.1, 292.7)), (False, 192, 55531, (36.0, 45.2, 48.1, 39.8)),
    (True, 64, 1024, (6.4, 8.0, 12.6)), (True, 176, 30705, (71.1, 84.3, 83.7)), (True, 604, 4608, (138.0, 115.4, 133.4)),
    (True, 1024, 5760, (415.3, 334.2, 305.1)), (True, 384, 57856, (541.3, 463.9, 423.4)), (True, 512, 2262, (60.2, 64.8, 86.2))])
def test_the_tile_of_a_product_is_a_fast_one(choice, cplx, n, B, us):
    columns = 2 * B if cplx else B
    tile = choice.product(n, 2 * n if cplx else n, ctypes.c_longlong(columns), 256, cplx)
    assert us[tile] <= 1.04 * min(us)


# ... of contractions without their sum, per tile (64 x 64, 128 x 128, 256 x 128) and slices.  The estimate has a standard
# deviation of 5 to 7 % over those it was fitted to.
@pytest.mark.parametrize("n,B,tile,slices,us", [
    (366, 8768, 0, 45, 29.5), (256, 16819, 0, 87, 26.4), (640, 3456, 0, 18, 28.4), (256, 4111, 0, 21, 11.5),
    (474, 3456, 0, 12, 19.0), (314, 648, 0, 1, 21.8), (768, 11264, 1, 29, 88.5), (1276, 9980, 1, 3, 271.2),
    (1428, 4032, 1, 3, 121.1), (2184, 4986, 1, 4, 335.8), (1018, 2052, 1, 5, 40.0), (1144, 15173, 1, 37, 266.9),
    (1024, 28608, 2, 49, 356.6), (1024, 6620, 2, 11, 96.0), (640, 6784, 2, 2, 348.1), (2196, 6400, 2, 9, 365.8)])
def test_estimates_of_contractions(choice, n, B, tile, slices, us):
    assert abs(choice.contraction_us(tile, slices, n, ctypes.c_longlong(B), 256) / us - 1) < 0.2


# Whatever the number of compute units: more workgroups never take less time.
@pytest.mark.parametrize("units", [8, 64, 256, 304])
def test_estimates_grow_with_the_work(choice, units):
    for tile in range(3):
        for n in (64, 200, 514):
            last = 0.0
            for slices in range(1, 120):
                us = choice.contraction_us(tile, slices, n, ctypes.c_longlong(512 * slices), units)
                assert us >= 0.98 * last
                last = us


# n = 228, B = 53484 was cut into 139 slices of 400 columns, of which 134 hold the columns: the others ran tiles for nothing.
@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("units", [64, 256, 304])
def test_the_slices_of_a_contraction_hold_its_columns_and_none_is_empty(choice, units, cplx):
    slices, cols = ctypes.c_int(), ctypes.c_longlong()
    shapes = [(228, 53484), (118, 115206), (34, 6513), (8192, 70000), (2, 256), (40, 2 ** 40)]
    shapes += [(n, 2 * n + 7 * n * k * k // 3) for n in range(34, 2300, 74) for k in range(24)]
    for n, B in shapes:
        choice.plan(n, ctypes.c_longlong(B), units, cplx, ctypes.byref(slices), ctypes.byref(cols))
        assert cols.value % 16 == 0 and (slices.value - 1) * cols.value < B <= slices.value * cols.value, (n, B)
        assert slices.value <= 256 and (cols.value <= 4096 or B > 4096 * 256 or slices.value * n * n * 4 > 2 ** 30)


# Restricted tiled sweeps: calls with every tile of a stage launched and with those that hold a free pair, in us, by the tiles, runs
# and steps of most of their stages.  Listed everywhere, the small ones were slower by up to 8 %.
@pytest.mark.parametrize("P,runs,per,active,all_us,listed_us", [
    (17, 1, 1, 2, 219, 229), (21, 1, 1, 2, 252, 267), (21, 2, 1, 2, 262, 271), (15, 14, 1, 4, 257, 265), (17, 63, 1, 6, 385, 403),
    (26, 47, 3, 8, 928, 977), (33, 32, 1, 10, 765, 795), (21, 32, 1, 12, 486, 510), (7, 25, 1, 5, 139.5, 143.5),
    (21, 141, 1, 2, 506, 427), (24, 32, 1, 8, 539, 458), (33, 43, 3, 10, 1389, 1293), (8, 63, 1, 2, 193, 164), (21, 22, 3, 10, 687, 663),
    (33, 21, 3, 25, 1930, 1770), (49, 63, 1, 8, 1518, 1300)])
def test_restricted_stages_are_listed_where_that_is_faster(choice, P, runs, per, active, all_us, listed_us):
    assert choice.listed(P, 256, ctypes.c_longlong(runs), ctypes.c_longlong(per), active) == (listed_us < all_us)


@pytest.mark.parametrize("P,all_us,listed_us", [(7, 417.5, 422.1), (8, 438.4, 443.6), (10, 671.7, 678.0), (14, 778, 785), (24, 1539, 1384),
                                                (33, 3375, 3287)])
def test_pairs_of_restricted_stages_are_listed_where_that_is_faster(choice, P, all_us, listed_us):
    assert choice.pairs_listed(P, 256) == (listed_us < all_us)
