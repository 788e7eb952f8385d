"""How many workgroups the quantisers of n = 256 .. 4096 run for any number of heads (csrc/bq_k12_grid.h)."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """#include "bq_k12_grid.h"
extern "C" long long per_head(long long rows, long long heads, int stores, int counts, int big, int f32)
{ return bq::quantiser_workgroups_per_head(rows, heads, {stores != 0, counts != 0, big != 0, f32 != 0}); }
"""


@pytest.fixture(scope="module")
def per_head(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    (d / "g.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_2509_09679_amd", "csrc"),
                    str(d / "g.cpp"), "-o", str(d / "g.so")], check=True)
    f = ctypes.CDLL(str(d / "g.so")).per_head
    f.argtypes, f.restype = [ctypes.c_longlong] * 2 + [ctypes.c_int] * 4, ctypes.c_longlong
    return f


# heads, rows per head, what (q: INT4 codes, y: fake-quantised INT2, h: with counts), groups above 128, float32 rows: measured us of a
# call with so many workgroups per head
MEASURED = [
    (129, 7, "q", 0, 0, {1: 12.2, 2: 16.2, 3: 16.4, 9: 29.4}), (129, 31, "q", 0, 0, {1: 33.6, 2: 30.3, 3: 26.8, 9: 42.2}),
    (171, 23, "q", 0, 0, {1: 28.0, 2: 27.0, 3: 31.4, 4: 31.8, 5: 36.5, 6: 40.1, 7: 43.6}),
    (171, 95, "q", 0, 0, {1: 89.6, 2: 68.7, 3: 74.8, 4: 66.4, 5: 69.2, 6: 74.2, 7: 74.6}),
    (171, 383, "q", 0, 0, {1: 338.0, 2: 236.5, 3: 254.4, 4: 213.1, 5: 205.8, 6: 216.5, 7: 205.0}),
    (171, 95, "q", 0, 1, {1: 91.7, 2: 78.1, 3: 90.0, 4: 79.9, 5: 85.8, 6: 89.7, 7: 88.3}),
    (171, 191, "q", 1, 0, {1: 270.8, 2: 183.6, 3: 197.9, 4: 159.4, 5: 158.8, 6: 168.2, 7: 154.2}),
    (171, 95, "y", 0, 0, {1: 96.9, 2: 76.4, 3: 85.2, 4: 76.0, 5: 79.6, 6: 89.5, 7: 86.8}),
    (400, 81, "q", 1, 0, {1: 165.7, 2: 163.9, 3: 153.2, 4: 163.2}), (400, 81, "y", 0, 0, {1: 137.9, 2: 146.9, 3: 136.1, 4: 149.2}),
    (171, 191, "h", 0, 0, {1: 204.2, 2: 152.7, 3: 171.7, 4: 142.5, 5: 144.2, 6: 156.1, 7: 146.0}),
    (200, 327, "q", 0, 0, {1: 291.8, 2: 211.7, 3: 224.3, 4: 209.9, 5: 196.3, 6: 201.2}),
    (257, 63, "q", 0, 0, {1: 84.3, 2: 76.1, 3: 70.6, 4: 74.5}), (257, 255, "q", 0, 0, {1: 305.7, 2: 259.3, 3: 221.4, 4: 221.7}),
    (300, 13, "q", 0, 0, {1: 28.6, 2: 31.9, 3: 37.1, 4: 43.7}), (300, 54, "q", 0, 0, {1: 76.1, 2: 70.8, 3: 67.7, 4: 74.2}),
    (300, 218, "q", 0, 0, {1: 271.7, 2: 229.7, 3: 206.0, 4: 203.4}), (300, 109, "q", 0, 1, {1: 165.0, 2: 166.1, 3: 153.7, 4: 151.7}),
    (300, 109, "y", 0, 0, {1: 161.0, 2: 148.9, 3: 134.0, 4: 138.1}), (300, 54, "q", 1, 0, {1: 108.1, 2: 97.2, 3: 87.8, 4: 91.9}),
    (340, 48, "q", 0, 0, {1: 69.7, 2: 67.2, 3: 66.7}), (400, 40, "q", 0, 0, {1: 61.7, 2: 70.3, 3: 73.9}),
    (400, 81, "q", 0, 1, {1: 149.0, 2: 167.6, 3: 155.2}), (511, 32, "q", 0, 0, {1: 56.8, 2: 68.0}),
]


@pytest.mark.parametrize("heads,rows,what,big,f32,times", MEASURED)
def test_the_choice_is_near_the_best_measured(per_head, heads, rows, what, big, f32, times):
    p = per_head(rows, heads, what in "yh", what == "h", big, f32)
    assert p in times and times[p] <= 1.05 * min(times.values()), p


@pytest.mark.parametrize("big", [0, 1])
@pytest.mark.parametrize("f32", [0, 1])
def test_no_head_count_leaves_units_idle(per_head, big, f32):
    # 100 rows and more per place: with every workgroup of a round of 512 taking equally long, the launch is at most 1.4 times as long
    # as its rows spread evenly (one workgroup per head for 257 heads: 1.99)
    for heads in range(1, 513):
        for rows in (512 * 100 // heads + 1, 512 * 350 // heads + 1):
            p = per_head(rows, heads, 0, 0, big, f32)
            assert 1 <= p <= rows
            w = heads * p
            rounds = w // 512 + (0 if w % 512 == 0 else 0.7 if w % 512 <= 256 else 1.0)
            assert -(-rows // p) * rounds <= 1.4 * rows * heads / 512, (heads, rows, p)


def test_one_head_and_divisors_keep_their_lines(per_head):
    for heads in (1, 2, 8, 32, 64, 128, 256):
        for blocks, counts, big, f32, want in ((1280, 0, 0, 0, 256), (3072, 1, 0, 0, 256), (2048, 0, 0, 0, 512), (4096, 1, 1, 1, 512),
                                               (1 << 17, 0, 0, 0, 512), (3 << 16, 0, 0, 0, 1280), (3 << 15, 0, 0, 1, 1280), (1 << 18, 0, 1, 0, 512)):
            rows = blocks // heads
            assert per_head(rows, heads, 0, counts, big, f32) == min(rows, want // heads)
    assert per_head(1, 512, 0, 0, 0, 0) == 1 and per_head(3, 1, 0, 0, 0, 0) == 3
