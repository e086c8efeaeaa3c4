"""The small-batch kernel's requests at 2 and 3 bits (csrc/fq_batch_at.h): two quantization groups of a row to a request,
a lane's 8 or 12 bytes of each at a time.  Walked as the kernel walks them, every one stays inside the weight it reads and the
run's rows are read whole (CPU only).  And the arithmetic by which a 3-bit block of 32 codes unpacks into the inputs' order, in
a copy here: that masks, shifts and exponents give exact differences; the kernel's own are checked in test_gpu_batch_narrow.py."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_12024_amd", "csrc")

DRIVER = r"""
#include "fq_batch_at.h"
extern "C" long walk(int N, int K, int bits, int n0, int nt, int kp_max, unsigned char *seen, long *missing)
{
    const uint32_t row_bytes = (uint32_t)K / 8 * bits, LB = batch_line_bytes(bits);
    const long whole = (long)N * row_bytes, base = (long)n0 * row_bytes;
    const uint32_t records = batch_run_bytes(row_bytes, nt, N - n0);
    const int KL = batch_line_inputs(bits), WAVES = 8, AHEAD = 2, piece = LB / 8;
    long bad = 0;
    for (int k0 = 0; k0 < K; k0 += kp_max) {
        const int kp = K - k0 < kp_max ? K - k0 : kp_max, lines = (kp + KL - 1) / KL;
        const uint32_t line0 = (uint32_t)k0 / 8 * bits;
        for (int wave = 0; wave < WAVES && wave < lines; wave++) {
            const int items = (lines - wave + WAVES - 1) / WAVES * nt;
            int it = 0, il = wave;
            for (int i = 0; i < items + 2 * AHEAD; i++) {
                for (int lane = 0; lane < 64; lane++)
                    for (int half = 0; half < 2; half++) {
                        const uint32_t at = batch_request(row_bytes, batch_lane_offset(row_bytes, lane & 15, lane >> 4, LB), it,
                                                          line0, il, LB) + LB / 2 * half;
                        if (at >= records)
                            continue;
                        const long addr = base + (long)at;
                        if (addr < 0 || addr + piece > whole || addr % 4 != 0 || at + piece > records)
                            bad++;
                        else if (i < items)
                            for (int b = 0; b < piece; b++)
                                seen[addr + b] = 1;
                    }
                il += WAVES;
                if (il >= lines)
                    il = wave, it++;
            }
        }
    }
    *missing = 0;
    const long last = n0 + nt * 16 < N ? n0 + nt * 16 : N;
    for (long p = base; p < last * row_bytes; p++)
        *missing += !seen[p];
    return bad;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("batch_narrow")
    src, lib = str(d / "walk.cpp"), str(d / "walk.so")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I", CSRC, "-o", lib, src])
    fn = ctypes.CDLL(lib).walk
    fn.restype = ctypes.c_long
    return fn


@pytest.mark.parametrize("bits", [2, 3])
def test_requests_stay_inside_the_weight(walk, bits):
    for (N, K, kp), nt in itertools.product([(16, 128, 4096), (1, 128, 4096), (33, 384, 4096), (37, 1152, 4096),
                                             (95, 2176, 2048), (96, 2176, 2048), (100, 4224, 4096), (61, 11008, 2048)],
                                            range(1, 7)):
        tiles = (N + 15) // 16
        for t0 in range(tiles - nt + 1):
            seen = (ctypes.c_ubyte * (N * K * bits // 8 + 1))()
            missing = ctypes.c_long()
            bad = walk(N, K, bits, t0 * 16, nt, kp, seen, ctypes.byref(missing))
            assert (bad, missing.value) == (0, 0), (N, K, t0, nt)


def test_the_last_offsets_do_not_wrap(walk):
    # the longest rows and runs: 6 tiles of 24576-byte rows (65536 inputs at 3 bits) and two requests ahead
    seen = (ctypes.c_ubyte * (112 * 65536 * 3 // 8 + 1))()
    missing = ctypes.c_long()
    assert walk(112, 65536, 3, 16, 6, 4096, seen, ctypes.byref(missing)) == 0 and missing.value == 0


def _half2(u):
    return np.array([u & 0xFFFF, u >> 16], dtype=np.uint16).view(np.float16)


def test_a_block_of_three_bit_codes_unpacks_in_order():
    # the kernel's masks, shifts and exponents, instruction by instruction: exact integers q - z, pairs of consecutive codes
    rng = np.random.default_rng(3)
    for _ in range(64):
        c, z = rng.integers(0, 8, 32), int(rng.integers(0, 8))
        v = []
        for j in range(3):
            w = 0
            for h in range(2):
                for p in range(5):
                    w |= int(c[10 * j + 5 * h + p]) << (16 * h + 3 * p)
                w |= ((int(c[30 + h]) >> j) & 1) << (16 * h + 15)
            v.append(w)
        z0, z3, z6 = z | 0xE400, (z << 3) | 0xD800, (z << 6) | 0xCC00
        got = []
        for w in v:
            lo, hi = (w & 0xFFFF) * 0x10001, (w >> 16) * 0x10001
            got += [((lo & 0x00380007) | 0x58006400, z0 | z3 << 16), ((lo >> 9 & 0x70000) | (lo & 0x1C0) | 0x64004C00, z6 | z0 << 16),
                    ((w & 0x70000) | (lo >> 9 & 0x38) | 0x64005800, z3 | z0 << 16), ((hi & 0x01C00038) | 0x4C005800, z3 | z6 << 16),
                    ((hi >> 9 & 0x00380007) | 0x58006400, z0 | z3 << 16)]
        last = (v[0] >> 15 & 0x10001) | (v[1] >> 14 & 0x20002) | (v[2] >> 13 & 0x40004)
        got.append((last | 0x64006400, z0 | z0 << 16))
        assert np.array_equal(np.concatenate([_half2(a) + _half2(n) for a, n in got]), (c - z).astype(np.float16))
