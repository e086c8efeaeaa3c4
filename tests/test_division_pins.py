"""The quantizers' shortened division (csrc/fq_div.h: a reciprocal, a product and one correction) against the IEEE
division that Sec. 2.2 Eq. (2) is pinned to (CPU only).  The header itself is compiled for the host, with
the few device names it uses mapped to their host counterparts, every one of which is rounded the same."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_12024_amd", "csrc")

STAND_IN = r"""
#include <cmath>
#include <cstdint>
#define __device__
#define __forceinline__ inline
static inline float __fdiv_rn(float a, float b) { return a / b; }
static inline float __fmul_rn(float a, float b) { return a * b; }
static inline float __fmaf_rn(float a, float b, float c) { return std::fmaf(a, b, c); }
static inline int __builtin_amdgcn_update_dpp(int, int v, int, int, int, bool) { return v; }
"""

DRIVER = r"""
#include "fq_div.h"
extern "C" void divide(const float *w, float s, float *out, long n)
{
    const Divisor by(s);
    for (long i = 0; i < n; i++)
        out[i] = by.of(w[i]);
}
// Pairs of an 11-bit w and a 24-bit s whose quotient lies within 64 units of the middle between two floats, the two
// next to T = n / 2 or n / 2 +- 2^-j: where the sum of the quotient and an integer zero point turns over.  |w 2^t - m S| <=
// 64 for a middle m of 25 or 26 bits is a distance of at most 2^-18 ulp; the quotient before its rounding is off by
// less than 2^-22.  Counts the pairs, and in *bad those whose result is not the IEEE quotient.
extern "C" long near_middles(int n_first, int n_last, long *bad)
{
    long found = 0;
    *bad = 0;
    for (int n = n_first; n <= n_last; n++)
        for (int j = 2; j <= 29; j++)
            for (int sign = -1; sign <= 1; sign += 2) {
                if (j == 2 && sign > 0)
                    continue; // j = 2: n / 2 itself
                const double T = n * 0.5 + (j == 2 ? 0.0 : sign * std::ldexp(1.0, -j));
                if ((double)(float)T != T)
                    continue;
                int ex;
                const uint64_t Ti = (uint64_t)std::ldexp(std::frexp(T, &ex), 24); // T = Ti 2^(ex - 24), 24 bits
                // middles in units of 2^(ex - 25): above, below; below a power of two floats are twice as dense
                const uint64_t middles[2] = {2 * Ti + 1, Ti == (1u << 23) ? 4 * Ti - 1 : 2 * Ti - 1};
                for (int q = 0; q < 2; q++) {
                    const uint64_t m = middles[q];
                    const int finer = q == 1 && Ti == (1u << 23);
                    for (uint64_t w = 1024; w < 2048; w++)
                        for (int t = 36; t <= 40; t++) {
                            const uint64_t a = w << t, down = a / m;
                            for (uint64_t S = down; S <= down + 1; S++) {
                                const uint64_t e = a > m * S ? a - m * S : m * S - a;
                                if (S < (1u << 23) || S >= (1u << 24) || e > 64)
                                    continue;
                                found++;
                                volatile float s = std::ldexp((float)S, 25 + finer - t - ex);
                                const float f = (float)w, want = f / s;
                                *bad += Divisor(s).of(f) != want || Divisor(s).of(-f) != -want;
                            }
                        }
                }
            }
    return found;
}
// Symmetric quantization, all of it up to powers of two: every largest magnitude (11 bits), width and weight that is
// not larger and not below 2^-12 of it.  Counts the weights, and in *bad those whose code differs from the division's.
extern "C" long symmetric(long *bad)
{
    long n = 0;
    *bad = 0;
    for (int a = 1024; a < 2048; a++)
        for (int bits = 2; bits <= 8; bits++) {
            const float amax = (float)a;
            volatile float s = (amax + amax) / (float)((1 << bits) - 2);
            const Divisor by(s);
            for (int e = 0; e <= 12; e++)
                for (int w = 1024; w < 2048; w++) {
                    const float f = std::ldexp((float)w, -e);
                    if (f > amax)
                        continue;
                    n++;
                    *bad += std::rint(by.of(f)) != std::rint(f / s);
                }
        }
    return n;
}
// Asymmetric quantization of random groups: a random range of halves, 64 weights of it each.
extern "C" long asymmetric(long groups, uint64_t seed, long *bad)
{
    long n = 0;
    *bad = 0;
    auto next = [&] {
        uint64_t z = (seed += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    };
    for (long g = 0; g < groups; g++) {
        const uint64_t r = next();
        const int bits = 2 + (int)(r % 7);
        const float hi = std::ldexp((float)(1024 + (r >> 8) % 1024), -(int)((r >> 20) % 12));
        const float lo = -std::ldexp((float)(1024 + (r >> 30) % 1024), -(int)((r >> 42) % 12));
        const float top = (float)((1 << bits) - 1);
        volatile float s = (hi - lo) / top;
        const Divisor by(s);
        const float z = std::fmin(std::fmax(std::rint(-lo / s), 0.0f), top);
        *bad += std::fmin(std::fmax(std::rint(by.of(-lo)), 0.0f), top) != z;
        for (int i = 0; i < 64; i++) {
            const uint64_t q = next();
            float f = std::ldexp((float)(1024 + q % 1024), -(int)((q >> 12) % 14));
            if (f > hi || (q >> 40 & 1))
                f = -f;
            if (f < lo)
                continue;
            n++;
            volatile float sum = by.of(f) + z, exact = f / s;
            exact = exact + z;
            *bad += std::rint(sum) != std::rint(exact);
        }
    }
    return n;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("div")
    os.mkdir(str(d / "hip"))
    for name, text in (("hip/hip_runtime.h", STAND_IN), ("driver.cpp", DRIVER)):
        with open(str(d / name), "w") as f:
            f.write(text)
    # (a processor without fused multiply-add rounds std::fmaf the same, only slower)
    fma = ["-mfma"] if " fma " in open("/proc/cpuinfo").read() else []
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fno-fast-math"] + fma +
                          ["-shared", "-fPIC", "-I", str(d), "-I", CSRC, "-o", str(d / "div.so"), str(d / "driver.cpp")])
    return ctypes.CDLL(str(d / "div.so"))


def _divide(lib, w, s):
    w = np.ascontiguousarray(w, dtype=np.float32)
    out = np.empty_like(w)
    p = ctypes.c_void_p
    lib.divide(w.ctypes.data_as(p), ctypes.c_float(s), out.ctypes.data_as(p), ctypes.c_long(w.size))
    return out


def _same(a, b):
    return np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(a[~np.isnan(a)], b[~np.isnan(b)])


def test_an_infinite_scale_divides_like_the_division(lib):
    # a group or row that holds an infinity has an infinite scale: its finite entries divide to 0, the infinite ones
    # to NaN
    w = np.array([0.0, -0.0, 1.0, -1.0, 65504.0, 2.0 ** -24, np.inf, -np.inf, np.nan], dtype=np.float32)
    with np.errstate(invalid="ignore"):
        want = w / np.float32(np.inf)
    assert _same(_divide(lib, w, np.inf), want)


def _count(fn, *args):
    fn.restype = ctypes.c_long
    bad = ctypes.c_long(-1)
    return fn(*args, ctypes.byref(bad)), bad.value


def test_quotients_next_to_the_middle_of_two_floats(lib):
    # every n / 2 that a code or a code less a zero point can turn over at
    found, bad = _count(lib.near_middles, ctypes.c_int(1), ctypes.c_int(1023))
    assert found > 1000 and bad == 0


def test_symmetric_codes_are_the_division_s(lib):
    n, bad = _count(lib.symmetric)
    assert n > 80000000 and bad == 0


def test_asymmetric_codes_are_the_division_s(lib):
    n, bad = _count(lib.asymmetric, ctypes.c_long(400000), ctypes.c_uint64(1))
    assert n > 10000000 and bad == 0
