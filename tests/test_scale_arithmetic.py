"""float32 scales: the short quotient and reciprocal sequences are the correctly rounded ones for every significand."""
import ctypes
import subprocess

import numpy as np
import pytest

import oracle

# m / 7 and 1 / s as the kernels form them (csrc/bq_cascade.h, scaled8), over all 2^23 significands; the hardware's estimate of 1 / s is
# within 1 ulp of it, so every float within that distance is tried.  Returns the number of wrong results; the significand of
# all ones, which the kernels send through the division, is counted apart.
SOURCE = r"""
#include <math.h>
#include <stdint.h>
#include <string.h>
static float f(uint32_t b) { float x; memcpy(&x, &b, 4); return x; }
static uint32_t u(float x) { uint32_t b; memcpy(&b, &x, 4); return b; }
long quotients(int e)
{
    const float k = 1.0f / 7.0f;
    long bad = 0;
    for (uint32_t m = 0; m < 1u << 23; ++m) {
        const float x = f((uint32_t)(127 + e) << 23 | m), q = x * k;
        if (fmaf(fmaf(-7.0f, q, x), k, q) != x / 7.0f) ++bad;
    }
    return bad;
}
long reciprocals(int e, long *all_ones)
{
    long bad = 0;
    *all_ones = 0;
    for (uint32_t m = 0; m < 1u << 23; ++m) {
        const float s = f((uint32_t)(127 + e) << 23 | m), want = 1.0f / s;
        int x;
        const double t = 1.0 / (double)s;
        frexp(t, &x);
        const double ulp = ldexp(1.0, x - 24);
        for (int d = -1; d <= 1; ++d) {
            const float r = f(u(want) + d);
            if (fabs((double)r - t) > ulp || fmaf(fmaf(-s, r, 1.0f), r, r) == want) continue;
            if (m == 0x7FFFFF) ++*all_ones; else ++bad;
        }
    }
    return bad;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("scale")
    (d / "s.c").write_text(SOURCE)
    subprocess.run(["gcc", "-O2", "-mfma", "-ffp-contract=off", "-shared", "-fPIC", str(d / "s.c"), "-o", str(d / "s.so"), "-lm"], check=True)
    L = ctypes.CDLL(str(d / "s.so"))
    L.quotients.restype = L.reciprocals.restype = ctypes.c_long
    return L


@pytest.mark.parametrize("e", [-90, -1, 0, 99])
def test_every_significand(lib, e):
    assert lib.quotients(e) == 0
    ones = ctypes.c_long()
    assert lib.reciprocals(e, ctypes.byref(ones)) == 0
    assert ones.value > 0  # why the kernels test for it


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [2, 4])
def test_float32_scales_bit_exact_over_significands_and_exponents(bits):
    # theta = 0 passes float32 rows through unchanged; group 8 at n = 8.  Values sit on and beside the rounding boundaries of the codes,
    # where a last bit of the reciprocal shows; a zero group, and exponents on both sides of the lines to the divisions (below
    # 2^-123 the reciprocal may overflow).
    gu = pytest.importorskip("gpu_util")
    rng = np.random.default_rng(77)
    m = np.concatenate([rng.integers(0, 1 << 23, 200000), np.full(2000, 0x7FFFFF), np.zeros(200, np.int64), np.full(200, 0x7FFFFE)])
    exps = np.concatenate([rng.integers(4, 254, len(m) // 2), rng.integers(30, 45, len(m) - len(m) // 2)])  # 2^-90 lies at 37
    amax = (exps.astype(np.uint32) << 23 | m.astype(np.uint32)).view(np.float32)
    amax[:4] = [0.0, np.float32(2.0**-123), np.float32(2.0**-90), np.float32(3e38)]
    qmax = (1 << (bits - 1)) - 1
    s = amax / np.float32(qmax)
    x = np.empty((len(m), 8), np.float32)
    x[:, 0] = amax
    for j in range(1, 8):
        edge = (np.float32(0.5 + (j % qmax)) * s).astype(np.float32)
        step = rng.integers(-1, 2, len(m))
        x[:, j] = np.minimum((edge.view(np.int32) + np.where(edge > 0, step, 0)).astype(np.int32).view(np.float32), amax) * rng.choice([-1.0, 1.0], len(m))
    th = np.zeros((1, 3, 4), np.float32)
    codes, scales = gu.run_fwd_quant(x, th, 8, 1, "f32", bits, 8, "f32")
    want_codes, want_scales = oracle.quantize(x, 8, bits, "f32")
    np.testing.assert_array_equal(scales.reshape(-1).view(np.uint32), want_scales.reshape(-1).view(np.uint32))
    np.testing.assert_array_equal(codes.reshape(-1), oracle.pack_codes(want_codes, bits).reshape(-1))
