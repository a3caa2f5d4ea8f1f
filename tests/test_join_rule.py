"""The rule by which a wave of a join's LDS write pass emits its matches, and by
which R payloads get room in LDS (csrc/join_rule.hpp), compiled for the host: the faster
side where both were timed, and the waves a compute unit keeps."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2312_00720_amd", "csrc")

SRC = """
#include "join_rule.hpp"
extern "C" int in_order(int cols, unsigned lanes, unsigned long long out, unsigned rows) {
    return gj::write_in_order(cols, lanes, out, rows);
}
extern "C" int stage(int cols, unsigned long long out, unsigned long long s_rows) {
    return gj::stage_payloads(cols, out, s_rows);
}
extern "C" int fits(unsigned long long lds, int waves) { return gj::staging_fits(lds, waves); }
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    src, so = d / "rule.cpp", d / "rule.so"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o",
                    str(so)], check=True)
    L = ctypes.CDLL(str(so))
    L.in_order.argtypes = [ctypes.c_int, ctypes.c_uint, ctypes.c_ulonglong, ctypes.c_uint]
    L.stage.argtypes = [ctypes.c_int, ctypes.c_ulonglong, ctypes.c_ulonglong]
    L.fits.argtypes = [ctypes.c_ulonglong, ctypes.c_int]
    return L


# payload columns of both sides, matches per S row, share of S rows with several -> in order
TIMED = [
    (2, 1.0001, 0.0001, False), (2, 1.1, 0.1, False), (2, 2, 1, False), (2, 4, 1, True), (2, 16, 1, True),
    (4, 1.0001, 0.0001, False), (4, 1.002, 0.002, True), (4, 1.1, 0.1, True), (4, 4, 1, True),
    (16, 1.0001, 0.0001, False), (16, 1.002, 0.002, True), (16, 2, 1, True), (16, 0.4, 0.1, True),
]


@pytest.mark.parametrize("cols,matches,share,want", TIMED)
def test_faster_side(rule, cols, matches, share, want):
    rows = 2048
    lanes = round(64 * (1 - (1 - share) ** (rows / 64)))
    if round(share * rows) == 0:
        lanes = 0
    assert bool(rule.in_order(cols, lanes, round(matches * rows), rows)) == want


def test_ends(rule):
    assert not rule.in_order(8, 0, 0, 0) and not rule.in_order(8, 0, 2048, 2048)
    assert rule.in_order(8, 64, 2 ** 40, 2 ** 32 - 1) == 0 and rule.in_order(8, 64, 2 ** 40, 65536) == 1


@pytest.mark.parametrize("waves,most", [(4, 160 * 1024 // 3), (8, 80 * 1024), (16, 156 * 1024)])
def test_staging_leaves_twelve_waves(rule, waves, most):
    assert rule.fits(most, waves) and not rule.fits(most + 8, waves) and rule.fits(8192, waves)


def test_staging_needs_output(rule):
    n = 1 << 24
    assert not rule.stage(2, 2 * n, n) and rule.stage(2, 3 * n, n) and rule.stage(2, 4 * n, n)
    assert not rule.stage(4, n + n // 2000, n) and rule.stage(4, n + n // 100, n) and not rule.stage(16, n // 2, n)
