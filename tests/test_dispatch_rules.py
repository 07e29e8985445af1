"""The host-side rules that pick a kernel form, compiled on their own (no GPU): the rule headers
hold plain C++."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2312_04429_amd", "csrc")


def _compiled(tmp_path_factory, name, code):
    d = tmp_path_factory.mktemp(name)
    src, out = str(d / "rule.cpp"), str(d / "rule.so")
    with open(src, "w") as f:
        f.write(code)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    src, "-o", out], check=True)
    return C.CDLL(out)


@pytest.fixture(scope="module")
def scan_rule(tmp_path_factory):
    lib = _compiled(tmp_path_factory, "scan", """
#include "lookup_rule.h"
extern "C" int blocks(long long tiles, int dp, int m) {
  return nv::resident_query_blocks(tiles, dp, m);
}
""")
    lib.blocks.argtypes = [C.c_longlong, C.c_int, C.c_int]
    return lib.blocks


# (rows, width, queries, us of the whole lookup with the row-resident scan, with two and with four
# query blocks per wave of the query-resident one), measured on one MI355X
SCANS = [
    (4000000, 768, 65, 1161, 1192, 1548), (4000000, 768, 128, 1489, 1261, 1597), (4000000, 768,
    129, 1625, 2406, 1582), (4000000, 768, 256, 2286, 2548, 1749), (4000000, 768, 272, 2403, 3813,
    3336), (4000000, 768, 400, 3162, 5071, 3445), (4000000, 768, 512, 3713, 5169, 3545), (1000000,
    768, 272, 670, 953, 867), (1000000, 768, 640, 1181, 1617, 1283), (1000000, 768, 1024, 1797,
    2620, 1778), (200000, 768, 144, 135, 173, 137), (200000, 768, 256, 176, 179, 144), (200000,
    768, 320, 215, 256, 240), (50000, 768, 256, 81, 91, 77), (50000, 768, 272, 111, 133, 134),
    (3000, 768, 129, 56, 52, 55), (3000, 768, 1024, 154, 80, 86), (20000, 768, 256, 66, 68, 60),
    (1000000, 640, 112, 342, 299, 374), (1000000, 640, 272, 564, 830, 733), (200000, 640, 224,
    139, 150, 121), (1000000, 512, 129, 322, 477, 332), (1000000, 512, 256, 438, 485, 341),
    (1000000, 512, 320, 525, 723, 645), (200000, 512, 112, 83, 81, 97), (200000, 512, 576, 219,
    272, 235), (4000000, 384, 144, 780, 1021, 982), (4000000, 384, 256, 1108, 1102, 1027),
    (1000000, 384, 144, 219, 275, 275), (1000000, 384, 272, 326, 502, 539), (200000, 384, 65, 55,
    67, 80), (3000, 384, 512, 68, 46, 50), (4000000, 256, 129, 518, 812, 784), (4000000, 256, 256,
    771, 862, 810), (1000000, 256, 144, 145, 222, 221), (200000, 256, 320, 80, 88, 91)]


@pytest.mark.parametrize("n,d,m,rows,two,four", SCANS)
def test_scan_choice_loses_nothing(n, d, m, rows, two, four, scan_rule):
    """No choice is slower than the row-resident scan by more than the timings' spread (2.5 %), and
    where the query-resident scan is clearly faster (by 12 % and more) it is taken."""
    pick = scan_rule(-(-n // 128), d, m)
    t = {0: rows, 2: two, 4: four}
    assert t[pick] <= 1.025 * rows
    assert t[pick] <= 1.12 * min(t.values())


def test_scan_choice_has_a_kernel(scan_rule):
    """Every width the rule names has an instance of the scan (multiples of 128 from 256 to 768)."""
    for d in range(128, 2049, 128):
        for m in (1, 64, 65, 128, 256, 257, 1024, 4096):
            for tiles in (0, 1, 24, 255, 256, 511, 512, 7813, 1 << 24):
                pick = scan_rule(tiles, d, m)
                assert pick in (0, 2, 4)
                assert pick == 0 or (256 <= d <= 768 and m > 64 and tiles > 0)
