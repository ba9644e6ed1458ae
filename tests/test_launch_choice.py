"""Host-side choices of the sweeps' launches (csrc/carousel_host.hpp), compiled for the host alone and compared with measured times."""
import ctypes
import os
import subprocess

import pytest

from paper_2106_00003_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "carousel_host.hpp"
using namespace givens;
extern "C" {
int wave64_strips(int n, long long B) { return wave64_bwd_strips(n, B); }
int unitary_width(long long B) { return unitary_fwd_width(2 * B, 1); }
int unitary_strips(long long B) { const int w = unitary_fwd_width(2 * B, 1); return unitary_fwd_strips((2 * B + w - 1) / w); }
int turned(int n, long long B) { return carousel_turned(n, B); }
}
"""


@pytest.fixture(scope="module")
def choice(tmp_path_factory):
    folder = tmp_path_factory.mktemp("launch_choice")
    source, library = str(folder / "choice.hip"), str(folder / "libchoice.so")
    with open(source, "w") as f:
        f.write(SOURCE)
    subprocess.run([build.hipcc_path(), "-std=c++17", "-O1", "-shared", "-fPIC", "--offload-arch=gfx950", "--offload-host-only",
                    "-I" + os.path.join(ROOT, "paper_2106_00003_amd", "csrc"), source, "-o", library], check=True)
    return ctypes.CDLL(library)


# Float64 backward calls in us with one strip per workgroup and row of sums, and with four: the choice is within 3 % of the faster.  By
# columns times n alone n = 136 was up to 8 % slower than with four, and n = 832 to 896 up to 10 % than with one.
@pytest.mark.parametrize("n,B,one,four", [
    (136, 112, 29.4, 31.3), (136, 192, 33.2, 30.9), (140, 256, 35.5, 32.6), (156, 160, 35.7, 34.3), (172, 128, 36.6, 36.6),
    (188, 256, 41.7, 42.3), (200, 160, 41.2, 42.6), (252, 192, 50.1, 54.4), (264, 256, 66.9, 72.9), (384, 256, 99.4, 101.6),
    (448, 256, 115.0, 117.0), (480, 224, 121.1, 123.7), (512, 192, 124.2, 131.6), (512, 256, 154.2, 134.3), (528, 256, 224.4, 251.3),
    (528, 272, 276.7, 250.9), (576, 256, 285.5, 272.9), (608, 224, 270.1, 284.9), (608, 256, 299.5, 288.2), (640, 192, 261.0, 298.1),
    (672, 192, 320.9, 314.7), (704, 160, 299.0, 329.0), (736, 160, 304.9, 343.1), (768, 160, 335.3, 357.4), (768, 192, 379.2, 359.7),
    (800, 128, 318.8, 369.0), (832, 128, 350.6, 384.7), (832, 160, 420.3, 388.0), (864, 128, 370.2, 398.9), (896, 112, 364.7, 412.6),
    (896, 128, 392.0, 417.2), (896, 160, 457.0, 420.1), (928, 128, 467.2, 444.2), (960, 96, 431.0, 438.5), (960, 128, 511.0, 444.6),
    (1024, 64, 334.0, 462.0), (1024, 128, 552.7, 475.6), (128, 128, 28.4, 24.1), (64, 4, 14.9, 14.6)])
def test_float64_rows_of_sums(choice, n, B, one, four):
    assert {1: one, 4: four}[choice.wave64_strips(n, ctypes.c_longlong(B))] <= 1.03 * min(one, four)


# Forward sweeps with eight slots per lane in us, with the table in the order of the angles and turned; strips of one wavefront (the staged
# sweep, which takes either), then of several, of which n = 1040 to 1232 with two columns and up to three strips per compute unit are up to 6 % slower turned.
@pytest.mark.parametrize("n,B,plain,turned", [
    (1024, 440, 113.0, 112.7), (1024, 512, 118.0, 117.9), (528, 513, 60.9, 60.7), (768, 1024, 92.3, 92.1), (768, 1030, 108.6, 107.3),
    (1024, 1030, 146.8, 143.6), (896, 1536, 135.5, 133.7), (1024, 1536, 156.4, 152.7), (896, 1600, 131.9, 129.4), (1024, 2040, 197.0, 191.1),
    (1040, 1, 237.2, 230.5), (1040, 640, 281.7, 235.5), (1040, 1200, 291.6, 306.8), (1040, 1536, 298.2, 309.8), (1040, 1560, 375.1, 314.1),
    (1072, 1400, 299.6, 316.6), (1104, 1100, 306.3, 324.6), (1104, 1536, 318.7, 327.5), (1104, 1700, 446.6, 359.2),
    (1168, 1400, 333.5, 346.3), (1168, 1536, 383.5, 368.1), (1232, 1200, 356.1, 364.2), (1232, 1400, 402.0, 385.8),
    (1264, 1025, 361.3, 343.1), (1264, 1200, 366.3, 370.7), (1264, 1300, 413.9, 395.2), (1328, 1200, 435.8, 410.8), (1536, 1200, 512.1, 468.0),
    (2048, 1, 499.4, 457.4), (2048, 1976, 995.1, 682.0), (3072, 64, 790.8, 722.4), (4096, 512, 1387.2, 1242.3)])
def test_turned_tables(choice, n, B, plain, turned):
    assert (turned if choice.turned(n, ctypes.c_longlong(B)) else plain) <= 1.015 * min(plain, turned)


# which of the sizes of tests/test_gpu_turned.py are turned, on both sides of every line
@pytest.mark.parametrize("n,B,expected", [(528, 512, 0), (528, 513, 1), (528, 768, 1), (528, 771, 1), (1024, 439, 0), (1024, 440, 1),
                                          (1024, 1021, 1), (1024, 1024, 1), (1024, 1025, 1), (1024, 1537, 1), (768, 1535, 1), (1008, 2007, 1),
                                          (1024, 2048, 1), (1024, 2049, 0), (1040, 1041, 0), (1040, 1561, 1), (1536, 30, 1), (3072, 257, 1), (4096, 131, 1)])
def test_sizes_that_are_turned(choice, n, B, expected):
    assert choice.turned(n, ctypes.c_longlong(B)) == expected


# Unitary forward calls in us: strips of two floats, one and four per workgroup, and of four floats; and as they were before tables
# were turned (a strip per workgroup), which some calls of few columns and some just above 1024 and 2048 were slower than.
@pytest.mark.parametrize("n,B,two_1,two_4,four_1,four_4,plain", [
    (128, 16, 49.0, 51.1, 66.7, 66.6, 50.4), (144, 16, 54.8, 58.0, 73.3, 73.4, 56.6), (144, 400, 56.8, 58.2, 73.8, 74.7, 58.2),
    (144, 1024, 60.8, 59.4, 75.6, 73.6, 64.0), (144, 1030, 68.0, 94.0, 75.3, 74.7, 72.3), (144, 1200, 68.7, 95.2, 76.0, 74.4, 73.4),
    (144, 1500, 78.5, 94.6, 76.3, 75.1, 83.6), (144, 2060, 114.1, 130.2, 87.6, 94.1, 85.4), (144, 3600, 162.9, 167.9, 120.7, 99.2, 121.4),
    (336, 128, 105.5, 108.1, 147.0, 147.1, 106.6), (336, 1200, 129.0, 179.3, 152.3, 146.7, 158.4),
    (336, 2400, 240.3, 257.0, 181.3, 180.5, 175.7), (336, 4090, 339.4, 336.6, 255.0, 193.0, 273.2),
    (512, 1024, 170.2, 167.3, 223.7, 215.4, 208.2), (512, 2060, 340.2, 383.1, 259.0, 257.7, 256.9),
    (640, 256, 204.9, 199.8, 265.6, 268.7, 202.3), (784, 2400, 585.8, 647.1, 405.3, 443.6, 447.7),
    (896, 1800, 622.1, 482.2, 445.5, 379.6, 858.4), (1024, 16, 285.6, 300.0, 411.7, 414.4, 308.4), (1024, 900, 323.5, 317.1, 431.1, 423.6, 504.1)])
def test_unitary_strips(choice, n, B, two_1, two_4, four_1, four_4, plain):
    wide = ctypes.c_longlong(B)
    us = {(2, 1): two_1, (2, 4): two_4, (4, 1): four_1, (4, 4): four_4}[choice.unitary_width(wide), choice.unitary_strips(wide)]
    assert us <= 1.035 * min(two_1, two_4, four_1, four_4, plain)
