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
