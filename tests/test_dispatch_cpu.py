"""CPU checks of csrc/dispatch.h, built alone with the host compiler: the order in which blocks take table entries, and the
rules that choose kernels."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_05451_amd", "csrc")

SHIM = r"""
#include "dispatch.h"
using namespace attn;
extern "C" {
int t_section_order(int block, int total) { return section_order(block, total); }
}
"""


@pytest.fixture(scope="module")
def D(tmp_path_factory):
    d = tmp_path_factory.mktemp("dispatch")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"),
                    "-o", str(d / "shim.so")], check=True)
    return ctypes.CDLL(str(d / "shim.so"))


@pytest.mark.parametrize("heads", [1, 2, 3, 4, 6, 8, 16, 32])
@pytest.mark.parametrize("lens", [[4096] * 16, [8192, 129, 700], [300] * 40, [257, 1025, 640, 64]])
def test_places_of_blocks_that_take_two_tiles(D, heads, lens):
    """Every place once; with a total that is dealt to the XCDs, every XCD has its share of the live places (those of a
    sequence's even tiles) and does not get them behind all of its empty ones."""
    max_tiles = sum(lens) // 128 + len(lens)
    tiles = [t for n in lens for t in range((n + 127) // 128 - 1, -1, -1)]              # a table: last tile first
    live = np.array([t % 2 == 0 for t in tiles] + [False] * (max_tiles - len(tiles)))
    total = max_tiles * heads
    places = np.array([D.t_section_order(b, total) for b in range(total)])
    assert sorted(places) == list(range(total))
    if total % 8:
        return
    took = live[places % max_tiles]
    for xcd in range(8):
        mine = places[xcd::8]
        assert mine.min() == xcd * (total // 8) and mine.max() == (xcd + 1) * (total // 8) - 1       # one section
        want = live[mine % max_tiles].sum()
        assert took[xcd::8].sum() == want
        used = (mine % max_tiles < len(tiles)).sum()            # half of a section's used entries, and one per sequence
        assert used / 2 - 1 <= want <= used / 2 + len(lens) * (1 + heads // 8)
