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
    return ctypes.CDLL(library)


# A contraction's workgroups reach the eight XCDs in turn; whatever their number, each XCD has consecutive ones of the list.
# n = 314, B = 15395 in 60 slices of 25 tiles: 70 us with the list handed out in turn, 38 so.
def test_every_xcd_has_a_consecutive_part_of_the_list(choice):
    for total in [*range(1, 130), 1500, 1504, 1530]:
        places = [choice.order(b, total) for b in range(total)]
        assert sorted(places) == list(range(total))
        for xcd in range(8):
            part = places[xcd::8]
            assert part == list(range(part[0], part[0] + len(part))) if part else total < 8
