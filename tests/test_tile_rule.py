"""The rule for the tiles of a partition pass in short chunks (csrc/scatter_rule.hpp),
compiled for the host: the fastest of the three shapes, or within 7% of it, at sizes
where all were timed, and the sizes at which it turns."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2312_00720_amd", "csrc")

SRC = """
#include "scatter_rule.hpp"
extern "C" int rows(unsigned long long n, unsigned nseg, int bits, int kb, unsigned row, int narrow) {
    const gj::TileShape t = gj::tile_shape(n, nseg, bits, kb, row, narrow != 0);
    return t.block * t.items;
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    src, so = d / "rule.cpp", d / "rule.so"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o",
                    str(so)], check=True)
    L = ctypes.CDLL(str(so))
    L.rows.argtypes = [ctypes.c_ulonglong, ctypes.c_uint, ctypes.c_int, ctypes.c_int, ctypes.c_uint, ctypes.c_int]
    return L


# rows, bits, key bytes, row bytes, all 4-byte data, us with tiles of 2048, 4096, 16384 rows
TIMED = [
    (1 << 20, 5, 4, 8, 1, 30, 33, 42), (1 << 20, 2, 4, 20, 1, 38, 38, 50), (1 << 20, 8, 8, 12, 0, 41, 40, 52),
    (1 << 21, 8, 4, 20, 1, 72, 62, 67), (1 << 21, 5, 4, 8, 1, 42, 36, 44), (1 << 21, 2, 4, 8, 1, 44, 34, 41),
    (1 << 21, 5, 8, 16, 0, 46, 50, 52), (1 << 21, 2, 8, 12, 0, 46, 43, 45), (1 << 21, 8, 8, 24, 0, 63, 66, 70),
    (2965820, 2, 4, 20, 1, 69, 64, 56), (2965820, 8, 4, 20, 1, 82, 74, 70), (2965820, 5, 8, 12, 0, 48, 58, 53),
    (1 << 22, 2, 4, 20, 1, 100, 76, 62), (1 << 22, 2, 8, 24, 0, 96, 102, 69), (1 << 22, 8, 4, 36, 1, 164, 137, 118),
    (1 << 22, 5, 8, 24, 0, 70, 90, 74), (1 << 22, 8, 4, 4, 1, 55, 54, 50),
    (5163608, 8, 4, 8, 1, 73, 70, 77), (5163608, 8, 4, 20, 0, 94, 88, 104), (5163608, 8, 4, 36, 1, 225, 187, 175),
    (5163608, 2, 4, 12, 1, 121, 83, 68), (5163608, 5, 4, 68, 0, 226, 206, 228), (5163608, 2, 4, 68, 0, 225, 187, 220),
    (5163608, 8, 4, 68, 0, 355, 304, 273), (6357300, 5, 4, 68, 0, 280, 258, 246),
    (5163608, 5, 8, 24, 0, 81, 102, 94),
    (6357300, 2, 8, 24, 0, 193, 195, 111), (6357300, 8, 4, 20, 1, 135, 118, 106), (6357300, 5, 4, 8, 1, 64, 71, 64),
    (1 << 23, 8, 4, 20, 1, 189, 156, 135), (1 << 23, 2, 8, 16, 0, 209, 201, 98),
]


@pytest.mark.parametrize("case", TIMED)
def test_fastest_tiles(rule, case):
    n, bits, kb, row, narrow, *us = case
    took = dict(zip((2048, 4096, 16384), us))[rule.rows(n, 1, bits, kb, row, narrow)]
    assert took <= 1.07 * min(us)


def test_turns(rule):
    r = rule.rows
    assert r(1 << 20, 1, 8, 4, 8, 1) == 2048 and r((1 << 20) + 1, 1, 8, 4, 8, 1) == 4096
    assert r(5 << 19, 256, 3, 4, 8, 1) == 4096 and r((5 << 19) + 1, 256, 3, 4, 8, 1) == 16384
    assert r(1 << 22, 1, 4, 4, 8, 1) == 16384 and r((1 << 22) + 1, 1, 4, 4, 8, 1) == 4096
    assert r(11 << 19, 1, 8, 4, 8, 1) == 4096 and r((11 << 19) + 1, 1, 8, 4, 8, 1) == 16384
    assert r(3 << 20, 128, 5, 4, 8, 1) == 4096 and r(3 << 20, 128, 5, 4, 12, 1) == 16384
    assert r(1 << 21, 1, 3, 8, 12, 0) == 2048 and r((1 << 21) + 1, 1, 3, 8, 12, 0) == 16384
    assert r(3 << 21, 256, 8, 8, 12, 0) == 2048 and r((3 << 21) + 1, 1, 8, 8, 12, 0) == 16384
    # a batch: by its rows and by the mean segment
    assert r(1 << 24, 4096, 8, 4, 8, 1) == 2048 and r(1 << 24, 1025, 8, 8, 16, 0) == 4096 and r(1 << 25, 300, 8, 4, 8, 1) == 16384
