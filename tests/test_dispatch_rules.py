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


class Plan(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("wide", "bm", "bn", "waves", "splits")]


@pytest.fixture(scope="module")
def stream_rule(tmp_path_factory):
    lib = _compiled(tmp_path_factory, "stream", """
#include "gemm_rule.h"
extern "C" nv::StreamPlan plan(long long M, int N, int K, int conv, int geglu, int ln, int rows_ok,
                               long long partial) {
  return nv::stream_plan({M, N, K, conv != 0, geglu != 0, ln != 0, rows_ok != 0, (size_t)partial});
}
extern "C" int forms() { return nv::WIDE_FORMS; }
""")
    lib.plan.restype = Plan
    lib.plan.argtypes = [C.c_longlong] + [C.c_int] * 6 + [C.c_longlong]

    def plan(M, N, K, conv, geglu=0, ln=0, rows_ok=1, partial=32 << 20):
        p = lib.plan(M, N, K, conv, geglu, ln, rows_ok, partial)
        assert -1 <= p.wide < lib.forms()
        per = -(-(K // 64) // p.splits)
        p.splits = -(-(K // 64) // per)  # as the launcher rounds it
        return p
    return plan


# (rows, columns, K, convolution, us of the small-tile kernels by their own rule, us of each form
# of the wide kernel), measured on one MI355X (graph-timed; the geometric mean of warm weights and
# weights streaming from HBM)
PRODUCTS = [
    (126, 320, 2880, 1, 10.8, (66.0, 47.7, 32.0, 31.0, 29.7, 22.4, 18.2, 17.5, 15.2)),
    (128, 320, 2880, 1, 10.8, (66.4, 47.8, 31.8, 31.0, 29.5, 22.4, 18.2, 17.5, 15.2)),
    (1408, 1280, 23040, 1, 108.0, (464.4, 358.4, 273.2, 206.0, 254.1, 147.5, 132.4, 185.1, 175.1)),
    (168, 320, 2880, 1, 11.0, (67.8, 48.4, 31.3, 30.9, 29.3, 22.4, 18.2, 17.6, 15.2)),
    (1152, 1280, 11520, 1, 53.5, (239.2, 180.5, 134.4, 106.4, 125.8, 76.1, 67.1, 95.0, 76.0)),
    (1232, 1280, 11520, 1, 50.9, (233.9, 176.3, 128.7, 100.4, 121.2, 73.0, 65.1, 91.3, 70.0)),
    (280, 320, 2880, 1, 11.4, (69.2, 49.2, 32.0, 31.0, 29.8, 22.5, 18.3, 17.6, 15.3)),
    (1024, 256, 4608, 1, 16.2, (101.6, 74.9, 47.1, 46.1, 44.4, 33.5, 26.5, 25.2, 22.3)),
    (320, 320, 2880, 1, 11.3, (69.4, 49.5, 31.9, 30.9, 29.8, 22.5, 18.3, 17.6, 15.2)),
    (640, 1280, 11520, 1, 36.3, (237.7, 181.8, 134.8, 106.8, 127.0, 76.3, 66.8, 52.0, 48.3)),
    (352, 320, 2880, 1, 11.4, (69.4, 49.6, 32.0, 31.0, 29.7, 22.5, 18.3, 17.6, 15.2)),
    (480, 320, 2880, 1, 11.6, (70.1, 50.0, 31.8, 31.4, 29.9, 22.9, 18.5, 17.8, 15.4)),
    (512, 320, 2880, 1, 11.7, (69.1, 49.4, 32.1, 31.0, 29.7, 22.6, 18.4, 17.6, 15.2)),
    (432, 320, 2880, 1, 11.6, (69.3, 49.6, 32.3, 31.1, 29.8, 22.6, 18.2, 17.6, 15.2)),
    (384, 320, 2880, 1, 11.6, (69.4, 49.4, 32.1, 30.9, 29.8, 22.5, 18.3, 17.5, 15.2)),
    (560, 320, 2880, 1, 11.8, (69.2, 49.4, 32.2, 31.1, 29.9, 22.6, 18.3, 17.6, 15.3)),
    (576, 320, 2880, 1, 12.0, (70.0, 50.1, 31.8, 31.4, 30.1, 22.8, 18.5, 17.8, 15.4)),
    (3072, 1280, 11520, 1, 106.9, (244.3, 191.8, 141.1, 108.6, 132.1, 126.7, 121.1, 149.4, 166.6)),
    (12288, 320, 320, 0, 13.8, (21.8, 15.0, 10.6, 10.8, 11.8, 10.4, 12.4, 17.8, 11.2)),
    (6144, 640, 11520, 1, 102.0, (238.0, 184.6, 133.0, 103.9, 124.5, 115.4, 111.2, 145.6, 150.6)),
    (80, 1280, 11520, 1, 17.2, (229.0, 174.3, 135.1, 102.5, 123.7, 73.4, 64.4, 48.1, 46.3)),
    (768, 1280, 5120, 0, 27.5, (109.8, 80.6, 60.6, 47.1, 54.7, 32.9, 29.7, 24.5, 20.7)),
    (12288, 256, 2304, 1, 26.6, (58.4, 44.2, 28.6, 28.1, 25.9, 28.4, 24.2, 43.6, 27.9)),
    (693, 400, 2048, 0, 11.3, (50.1, 35.4, 23.0, 22.2, 21.4, 15.7, 13.2, 12.2, 10.1)),
    (640, 640, 5760, 1, 21.3, (121.8, 87.5, 61.5, 53.3, 52.2, 38.0, 30.8, 27.0, 25.6)),
    (16384, 640, 640, 0, 29.4, (32.4, 24.1, 23.3, 29.6, 28.2, 27.2, 28.3, 54.5, 32.5)),
    (8192, 3840, 1280, 0, 112.3, (87.7, 96.2, 93.8, 117.6, 101.0, 123.4, 172.8, 240.8, 189.4)),
    (616, 2560, 768, 0, 10.6, (27.1, 19.6, 13.2, 13.2, 11.8, 9.7, 8.3, 14.7, 8.9)),
    (4096, 320, 2880, 1, 26.6, (70.8, 50.6, 31.8, 31.6, 30.4, 23.3, 19.4, 18.5, 21.4)),
    (5376, 3840, 1280, 0, 78.0, (78.8, 64.5, 63.6, 79.2, 75.8, 83.4, 114.5, 166.0, 126.8)),
    (640, 1152, 384, 0, 5.7, (20.6, 14.5, 9.7, 10.1, 8.5, 7.5, 6.4, 7.1, 5.3)),
    (1024, 1280, 23040, 1, 76.3, (473.6, 371.9, 274.4, 204.6, 253.4, 145.9, 130.7, 101.0, 147.2)),
    (1232, 768, 2048, 0, 13.5, (49.4, 36.1, 25.2, 22.8, 23.1, 16.3, 13.3, 12.7, 10.7)),
    (576, 256, 2304, 1, 11.4, (57.7, 42.4, 27.1, 26.7, 25.1, 19.6, 15.7, 15.6, 13.1)),
    (6336, 960, 320, 0, 16.1, (21.4, 15.2, 13.6, 18.7, 12.5, 14.7, 15.2, 27.8, 15.3)),
    (768, 1280, 1280, 0, 10.1, (36.4, 26.4, 17.8, 17.2, 16.2, 12.1, 10.3, 10.2, 8.3)),
    (7040, 640, 11520, 1, 149.6, (236.9, 180.1, 137.2, 106.9, 140.2, 123.6, 155.8, 186.9, 183.2)),
    (80, 256, 2304, 1, 10.5, (53.0, 39.9, 25.9, 26.0, 24.3, 18.9, 15.4, 15.2, 12.9)),
    (36864, 640, 1280, 0, 91.5, (81.0, 86.1, 72.3, 91.2, 72.4, 80.5, 88.2, 148.0, 111.1)),
    (19712, 1152, 384, 0, 37.8, (44.8, 44.6, 34.2, 46.5, 34.2, 40.9, 37.7, 96.8, 49.5)),
    (1152, 320, 2880, 1, 16.9, (70.5, 50.3, 32.0, 31.5, 30.3, 22.8, 18.6, 17.8, 15.6)),
    (24576, 320, 2880, 1, 74.6, (73.0, 53.1, 51.9, 63.0, 68.2, 54.7, 67.0, 98.6, 76.2)),
    (512, 1280, 23040, 1, 51.2, (478.2, 379.4, 262.8, 205.5, 251.2, 147.1, 129.0, 98.5, 93.4)),
    (231, 1280, 768, 0, 7.4, (26.1, 19.0, 12.8, 12.8, 11.3, 9.3, 7.8, 8.2, 6.4)),
    (720, 256, 2304, 1, 11.4, (57.6, 42.4, 27.2, 26.8, 25.2, 19.8, 15.8, 15.6, 13.2)),
    (1536, 1280, 23040, 1, 120.3, (476.2, 378.9, 275.1, 207.1, 258.0, 149.3, 133.9, 186.9, 179.7)),
    (4608, 1280, 5120, 0, 79.0, (116.5, 92.2, 82.9, 98.8, 74.5, 87.4, 87.5, 121.1, 116.8)),
    (4608, 256, 2304, 1, 23.5, (58.8, 43.4, 27.5, 27.5, 25.6, 20.2, 16.4, 29.6, 18.5)),
    (32768, 640, 2560, 0, 156.3, (141.3, 115.8, 112.8, 130.5, 124.9, 134.4, 145.8, 226.6, 184.3)),
    (140, 256, 2304, 1, 10.8, (55.0, 40.7, 26.5, 26.5, 24.6, 19.4, 15.5, 15.4, 13.0)),
    (385, 768, 768, 0, 7.5, (26.7, 19.3, 12.8, 12.9, 11.3, 9.3, 7.8, 8.2, 6.3)),
    (28672, 320, 320, 0, 29.6, (25.9, 18.5, 17.9, 22.3, 21.1, 20.6, 23.4, 42.2, 23.2)),
    (4608, 1280, 1280, 0, 28.6, (41.2, 30.5, 28.0, 35.9, 24.4, 29.9, 26.6, 45.7, 32.1)),
    (1152, 1280, 2560, 0, 22.0, (59.4, 45.3, 34.2, 27.9, 31.5, 19.5, 18.2, 27.6, 19.8)),
    (10240, 320, 1280, 0, 25.5, (41.3, 29.7, 22.2, 19.3, 19.6, 20.8, 18.5, 28.1, 21.6)),
    (65536, 1920, 640, 0, 260.4, (241.4, 262.0, 245.7, 313.1, 248.9, 278.9, 295.7, 603.1, 335.1)),
    (4096, 512, 384, 0, 8.8, (21.6, 16.3, 11.4, 11.2, 9.9, 8.3, 7.3, 12.9, 7.9)),
    (1024, 512, 64, 0, 4.2, (13.8, 10.5, 7.4, 7.6, 6.0, 5.6, 4.8, 6.0, 4.0)),
    (16384, 256, 192, 0, 10.6, (18.8, 14.2, 10.3, 10.3, 8.9, 9.9, 9.0, 21.8, 10.5)),
    (16384, 384, 64, 0, 9.7, (16.9, 12.2, 10.3, 14.9, 9.0, 11.6, 10.2, 24.3, 12.1)),
    (256, 128, 1152, 1, 10.3, (37.4, 27.2, 18.0, 18.1, 16.2, 13.2, 10.7, 11.2, 8.8)),
    (16384, 64, 1152, 1, 12.6, (40.3, 30.0, 19.7, 20.1, 17.9, 15.5, 12.0, 11.8, 10.2)),
    (8192, 128, 2304, 1, 18.3, (61.5, 45.4, 29.0, 28.9, 26.8, 21.9, 17.2, 17.9, 14.8)),
    (16, 768, 256, 0, 4.5, (11.8, 9.2, 6.6, 7.3, 5.8, 5.6, 4.8, 5.8, 4.3)),
    (128, 512, 192, 0, 4.8, (13.8, 10.4, 8.3, 8.6, 6.8, 6.1, 5.2, 6.2, 4.2)),
    (2048, 384, 128, 0, 4.9, (17.1, 11.7, 8.1, 8.4, 6.7, 6.1, 5.2, 6.2, 4.4)),
    (16384, 64, 1152, 1, 12.5, (40.7, 30.0, 19.5, 20.1, 17.9, 15.5, 12.0, 11.7, 10.2)),
]


@pytest.mark.parametrize("M,N,K,conv,small,wide", PRODUCTS)
def test_product_choice_loses_nothing(M, N, K, conv, small, wide, stream_rule):
    """No choice is slower than the small-tile kernels by more than 8 % (the spread of the cost
    estimates), nor than the fastest form by more than 15 %."""
    p = stream_rule(M, N, K, conv)
    t = small if p.wide < 0 else wide[p.wide]
    assert t <= 1.08 * small
    assert t <= 1.15 * min(small, *wide)


def test_wide_forms_are_given_up_only_for_a_split(stream_rule):
    """A product the wide forms take goes to the small tiles only where those do split K: the
    estimate that decides is the split's."""
    wide = split = 0
    for conv in (0, 1):
        for C1 in (64, 128, 256, 320, 512, 640, 1280, 2560):
            for K in ((9 * C1,) if conv else (C1, 4 * C1)):
                for N in (64, 256, 320, 640, 960, 1280, 2560, 3840):
                    for M in [int(64 * 1.09 ** i) for i in range(0, 92)]:
                        for partial in (0, 32 << 20, 1 << 30):
                            p = stream_rule(M, N, K, conv, partial=partial)
                            if p.wide < 0:
                                assert p.splits >= 2, (M, N, K, conv, partial)
                                split += 1
                            else:
                                wide += 1
    assert wide and split


def test_products_that_cannot_split(stream_rule):
    """Folded LayerNorm and GEGLU keep all of K in one workgroup; GEGLU takes the forms that pair
    its quads in registers; without the row-staged epilogue no wide form runs."""
    for M in (1, 77, 512, 2048, 8192, 65536):
        for N, K in ((320, 320), (1280, 1280), (5120, 640), (10240, 1280)):
            assert stream_rule(M, N, K, 0, ln=1).splits == 1
            g = stream_rule(M, N, K, 0, geglu=1, ln=1)
            assert g.splits == 1
            if -(-M // 128) * -(-N // 128) > 320:
                assert g.wide >= 0 and (g.bm, g.bn) in ((256, 256), (128, 128))
            else:  # the wide forms would leave CUs without a tile
                assert g.wide == -1
            for ln in (0, 1):
                p = stream_rule(M, N, K, 0, ln=ln, rows_ok=0)
                assert p.wide == -1 and (p.splits == 1 or not ln)


class Args(C.Structure):
    """The fields of a product that the row-staged epilogue's gate reads."""
    _fields_ = ([("M", C.c_longlong), ("rows_div", C.c_longlong), ("vt_ld", C.c_longlong),
                 ("vt_div", C.c_longlong), ("vt_stride", C.c_longlong)] +
                [(n, C.c_void_p) for n in ("out", "rowvec", "residual", "vt")] +
                [(n, C.c_int) for n in ("N", "ldo", "ld_res", "vt_col0", "vec_ok", "out_f32", "geglu")])


def test_row_epilogue_gate(tmp_path_factory):
    """What the row-staged epilogue cannot do goes elsewhere: transposed columns with a row vector
    (it adds none to them) or with GEGLU, float32 outputs, and anything off its 16-byte pieces."""
    lib = _compiled(tmp_path_factory, "gate", """
#include "gemm_rule.h"
struct Args {
  long long M, rows_div, vt_ld, vt_div, vt_stride;
  void *out, *rowvec, *residual, *vt;
  int N, ldo, ld_res, vt_col0, vec_ok, out_f32, geglu;
};
extern "C" int ok(const Args* a) { return nv::row_epilogue_ok(*a); }
""")
    base = dict(M=512, N=960, ldo=640, ld_res=640, vec_ok=1, out=0x1000, rows_div=1)
    vt = dict(vt=0x2000, vt_col0=640, vt_ld=512, vt_div=256, vt_stride=256)
    ok = lambda **over: bool(lib.ok(C.byref(Args(**dict(base, **over)))))
    assert ok() and ok(**vt) and ok(residual=0x3000) and ok(rowvec=0x4004, rows_div=256)
    assert ok(geglu=1) and ok(residual=0x3000, **vt)
    assert not ok(rowvec=0x4000, rows_div=256, **vt)
    assert not ok(geglu=1, **vt)
    for bad in (dict(vec_ok=0), dict(out_f32=1), dict(M=1 << 31), dict(N=956), dict(ldo=644),
                dict(out=0x1008), dict(residual=0x3008), dict(residual=0x3000, ld_res=644),
                dict(geglu=1, N=944), dict(rowvec=0x4000, rows_div=1 << 31)):
        assert not ok(**bad), bad
    for bad in (dict(M=511), dict(vt=0x2008), dict(vt_col0=644), dict(vt_ld=508), dict(vt_div=252),
                dict(vt_stride=252)):
        assert not ok(**dict(vt, **bad)), bad
