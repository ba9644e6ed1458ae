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
