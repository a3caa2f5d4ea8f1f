"""The rule that gives a partition pass long chunks and whole lines or short chunks
and the wide kernel (csrc/scatter_rule.hpp), compiled for the host: the LDS limits of
the line shapes, and the faster side at the sizes where both were timed."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2312_00720_amd", "csrc")

SRC = """
#include "scatter_rule.hpp"
extern "C" int chunks(unsigned long long n, unsigned nseg, int bits, unsigned row, int narrow, int aligned) {
    return gj::long_chunks(n, nseg, bits, row, narrow != 0, aligned != 0);
}
extern "C" int shape(int bits, unsigned row, int narrow) {
    const gj::LineShape s = gj::line_shape(bits, row, narrow != 0);
    return s.items * 100 + s.rows;
}
extern "C" unsigned long long lds(int bits, unsigned row, int narrow) {
    const gj::LineShape s = gj::line_shape(bits, row, narrow != 0);
    return s.items ? gj::line_lds_bytes(1u << bits, s.rows, row, 1024u * s.items, narrow ? 4 : 8) : 0;
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
    L.chunks.argtypes = [ctypes.c_ulonglong] + [ctypes.c_uint, ctypes.c_int, ctypes.c_uint, ctypes.c_int, ctypes.c_int]
    L.lds.restype = ctypes.c_ulonglong
    return L


def test_shapes_fit_the_lds(rule):
    for narrow in (0, 1):
        for bits in range(1, 9):
            for row in range(8, 140, 4):
                s = rule.shape(bits, row, narrow)
                if s:
                    assert (1 << bits) * (s % 100) <= 4096 and rule.lds(bits, row, narrow) <= 160 * 1024 - 128
    # the widest rows whose carry fits
    assert rule.shape(8, 24, 1) and not rule.shape(8, 28, 1)
    assert rule.shape(7, 56, 1) and not rule.shape(7, 60, 1)
    assert rule.shape(8, 12, 0) and not rule.shape(8, 16, 0)
    assert rule.shape(7, 36, 0) and not rule.shape(7, 40, 0)


# log2 of the output bytes, bytes a row, 4-byte data only, bits, segments -> long chunks
TIMED = [
    (28, 20, 1, 7, 1, False), (29, 20, 1, 7, 1, True), (29, 12, 1, 4, 1, True), (32, 12, 1, 8, 1, True),
    (29, 20, 1, 3, 1, False), (30, 8, 1, 2, 1, False), (32, 8, 1, 2, 1, False), (32, 12, 1, 1, 1, False),
    (32, 12, 1, 3, 1, True),                               # few bits: the runs split few lines
    (31, 20, 0, 8, 1, False), (31, 16, 0, 5, 1, False), (31, 20, 0, 4, 1, False), (32, 8, 0, 4, 1, False),
    (31, 16, 0, 7, 1, True), (32, 32, 0, 5, 1, True), (31, 8, 0, 6, 1, True), (30, 16, 0, 7, 1, False),
    (29, 28, 1, 8, 1, False), (30, 36, 1, 8, 1, False),    # no room for the carry
    (31, 28, 1, 8, 1, True), (32, 36, 1, 8, 1, True), (31, 40, 0, 7, 1, False),
    (31, 16, 0, 8, 256, False), (32, 16, 0, 8, 256, False), (31, 32, 1, 8, 256, False),
    (31, 12, 1, 7, 128, True), (31, 12, 1, 7, 257, False),
]


@pytest.mark.parametrize("case", TIMED)
def test_faster_side(rule, case):
    lg, row, narrow, bits, nseg, want = case
    n = 2 ** lg // row + 12345
    assert bool(rule.chunks(n, nseg, bits, row, narrow, 1)) == want
    assert not rule.chunks(n, nseg, bits, row, narrow, 0)  # 16-byte stores need aligned columns
