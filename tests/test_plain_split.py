"""How the backward pass splits a batch on a flagged plan (csrc/bq_plain_split.h): every row once, and float32 sums no less exact than
those of the kernel for any n."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """#include "bq_plain_split.h"
extern "C" void grown(int u, long long tiles, int parts, long long rows, int n, int heads, long long *out)
{ const bq::PlainSplit g = bq::grown_split({u, tiles, parts}, rows, n, heads); out[0] = g.rows_per_tile; out[1] = g.tiles; out[2] = g.parts; }
"""


@pytest.fixture(scope="module")
def grown(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    (d / "s.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_2509_09679_amd", "csrc"),
                    str(d / "s.cpp"), "-o", str(d / "s.so")], check=True)
    f = ctypes.CDLL(str(d / "s.so")).grown
    f.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int,
                  ctypes.POINTER(ctypes.c_longlong)]

    def call(u, tiles, parts, rows, n, heads):
        out = (ctypes.c_longlong * 3)()
        f(u, tiles, parts, rows, n, heads, out)
        return tuple(out)

    return call


def _general(rows, n, heads):  # bwd_geometry of csrc/bq_generic.hip
    u = max(1, 1024 // n)
    tiles = -(-rows // u) * heads
    k = n.bit_length() - 1
    cap = (32 << 20) // (heads * k * (n // 2) * 4)
    cap = max(cap - cap % heads, 8 * heads)
    return u, tiles, max(1, min(tiles, 512, cap))


def _rounding(rows, heads, u, parts, once):
    """Sum over the additions of a head's float32 sums of the squared number of rows in the result, per angle: what the variance of the
    accumulated rounding is proportional to for rows of equal size.  once: a tile's rows are added without rounding."""
    tiles = -(-rows // u)
    per = -(-parts // heads)
    total = 0.0
    for p in range(per):
        mine = tiles // per + (p < tiles % per)
        for t in range(mine):
            first = 1 if t == 0 else 0
            if not once:  # the first addition of a tile is to zero, and so is the first tile's to its slice
                total += sum(r for r in range(2, u + 1))
            if once and u > 1 or not first:
                total += (t + 1) * u
    return total


@pytest.mark.parametrize("n,heads", [(256, 1), (256, 16), (512, 1), (512, 8), (1024, 1), (1024, 2), (2048, 1), (2048, 2), (4096, 1), (8192, 1)])
def test_no_less_exact_than_the_general_pass(grown, n, heads):
    for rows in (1, 2, 100, 256, 257, 300, 341, 342, 511, 512, 513, 700, 1024, 1025, 2047, 2049, 5000, 20000, 100000):
        u, tiles, parts = _general(rows, n, heads)
        gu, gt, gp = grown(u, tiles, parts, rows, n, heads)
        assert gt == -(-rows // gu) * heads and 1 <= gp <= min(parts, gt)  # every row, and the slices the workspace holds
        assert gu * n <= 8192  # with the gradient 64 KB of LDS
        assert _rounding(rows, heads, gu, gp, True) <= _rounding(rows, heads, u, parts, False) * 1.01, (rows, (u, parts), (gu, gp))
