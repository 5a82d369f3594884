"""Where the products' and convolutions' 16-byte loads lie (csrc/row_pieces.h), walked on the host: what a GPU test cannot see, as
memory behind a tensor is as readable as the tensor and the kernels clear what a row does not hold."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1705_09864_amd", "csrc")
SOURCE = """
#define __host__
#define __device__
#define __forceinline__ inline
#include "row_pieces.h"
extern "C" unsigned back(int segment, int piece, int dwords) { return bmx::piece_back(segment, piece, dwords); }
extern "C" int meet(unsigned run, int segment) { return bmx::runs_meet(run, [&](unsigned x) { return x / (2 * run); }, segment); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_pieces")
    src, so = str(d / "pieces.cpp"), str(d / "pieces.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", so])
    return ctypes.CDLL(so)


def test_pieces_stay_inside_their_row(lib):
    """Rows of every length: 16 bytes from inside the row (its 16-byte slot where it is shorter), every dword of the row in the piece that
    stands for it, at the place that the kernels take it from, and no offset below zero with the 16 bytes that the kernels add."""
    for dwords in list(range(1, 150)) + [255, 256, 257, 4095, 4096]:
        slot = max(dwords, 4)
        for segment in range(-(-dwords // 16)):
            for piece in range(4):
                first = 16 * segment + 4 * piece  # of the row's dwords, were the row longer
                back = lib.back(segment, piece, dwords)
                start = 4 * first - back
                assert 0 <= start and start + 16 <= 4 * slot, (dwords, segment, piece)
                assert 16 + 16 * piece - back >= 0 and back % 4 == 0
                if first + 4 <= dwords:
                    assert back == 0
                elif first < dwords and dwords >= 4:  # the row's last 16 bytes: its last dwords - first ones are the piece's
                    assert start == 4 * (dwords - 4)
                elif first < dwords:
                    assert start == 0


@pytest.mark.parametrize("run", list(range(1, 40)) + [63, 64, 65, 99])
@pytest.mark.parametrize("rows", [1, 2, 3, 5, 7])
def test_segments_that_two_runs_meet_in(lib, run, rows):
    words = rows * run
    for segment in range(-(-words // 8)):
        meets = False
        for first in range(8 * segment, min(8 * segment + 8, words), 2):
            meets |= first + 1 >= words or first // run != (first + 1) // run
        assert bool(lib.meet(run, segment)) >= meets, (run, rows, segment)  # (a segment too many only costs time:
        if words % 8 == 0 or segment + 1 < -(-words // 8):                  # the last, behind whose row a run would go on)
            assert bool(lib.meet(run, segment)) == meets, (run, rows, segment)
