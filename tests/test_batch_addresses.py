"""Every weight request of the small-batch kernel (csrc/fq_batch.hip) stays inside the weight it reads, and its
division of a launch gives every tile to one workgroup and no workgroup far too many (CPU only).

The kernel's address and division rules are plain integer code (csrc/fq_batch_at.h), compiled for the host here.  The
requests of a run -- every wavefront, line, lane and half line, and the requests ahead past the last tile -- are
walked as the kernel walks them.  A lane whose offset is below the descriptor's size reads 16 bytes at that
offset; one whose offset is not reads nothing.  (The scalar offset is no part of the range check: the rule
must hold without it, and the kernel passes none.)"""
import ctypes
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_12024_amd", "csrc")

DRIVER = r"""
#include "fq_batch_at.h"
// Walks one run of nt tiles from row n0 of an N x K weight at `bits`; panels of kp inputs.  Returns the number of
// reads that leave the weight, and counts in *missing the 16-byte pieces of the run's rows that nobody read.
extern "C" long walk(int N, int K, int bits, int n0, int nt, int kp_max, unsigned char *seen, long *missing)
{
    const uint32_t row_bytes = (uint32_t)((long)K * bits / 8);
    const long whole = (long)N * row_bytes, base = (long)n0 * row_bytes;
    const uint32_t records = batch_run_bytes(row_bytes, nt, N - n0);
    const int KL = 1024 / bits, WAVES = 8, AHEAD = 2;
    long bad = 0;
    for (int k0 = 0; k0 < K; k0 += kp_max) {
        const int kp = K - k0 < kp_max ? K - k0 : kp_max, lines = (kp + KL - 1) / KL;
        const uint32_t line0 = (uint32_t)((long)k0 * bits / 8);
        for (int wave = 0; wave < WAVES; wave++) {
            if (lines <= wave)
                continue; // no line of this panel: no request
            const int items = (lines - wave + WAVES - 1) / WAVES * nt;
            int it = 0, il = wave;
            for (int i = 0; i < items + 2 * AHEAD; i++) {
                for (int lane = 0; lane < 64; lane++)
                    for (int half = 0; half < 2; half++) {
                        const uint32_t at = batch_request(row_bytes, batch_lane_offset(row_bytes, lane & 15, lane >> 4), it,
                                                          line0, il) + 64 * half;
                        if (at >= records)
                            continue;
                        const long addr = base + (long)at;
                        if (addr < 0 || addr + 16 > whole)
                            bad++;
                        else if (i < items)
                            seen[addr / 16] = 1;
                    }
                il += WAVES;
                if (il >= lines)
                    il = wave, it++;
            }
        }
    }
    *missing = 0;
    const long last = n0 + nt * 16 < N ? n0 + nt * 16 : N;
    for (long p = base / 16; p < last * row_bytes / 16; p++)
        *missing += !seen[p];
    return bad;
}
extern "C" int tile_cost(int blocks, int K, int bits) { return batch_tile_cost(blocks, K, bits); }
extern "C" int panel_of(int blocks) { return batch_panel(blocks); }
// The tiles of each entry that share i of `shares` takes: out[2 * (i * count + e)] .. out[2 * (i * count + e) + 1].
extern "C" void divide(int count, const int *N, const int *K, const int *bits, int blocks, int shares, int *out)
{
    uint32_t all = 0;
    for (int e = 0; e < count; e++)
        all += (uint32_t)((N[e] + 15) / 16) * batch_tile_cost(blocks, K[e], bits[e]) + BATCH_START_COST;
    for (int i = 0; i < shares; i++) {
        uint32_t begin = 0;
        for (int e = 0; e < count; e++) {
            const int tiles = (N[e] + 15) / 16, cost = batch_tile_cost(blocks, K[e], bits[e]);
            for (int h = 0; h < 2; h++)
                out[2 * (i * count + e) + h] = batch_first_tile(batch_share(all, i + h, shares), begin, cost, tiles);
            begin += (uint32_t)tiles * cost + BATCH_START_COST;
        }
    }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("batch_at")
    src, lib = str(d / "walk.cpp"), str(d / "walk.so")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I", CSRC, "-o", lib, src])
    return ctypes.CDLL(lib)


@pytest.fixture(scope="module")
def walk(lib):
    lib.walk.restype = ctypes.c_long
    return lib.walk


@pytest.mark.parametrize("bits", [4, 8, 16])
def test_requests_stay_inside_the_weight(walk, bits):
    # whole and partial last tiles, alone and at the end of a run; one group, odd and even numbers of groups; several
    # panels of x (4096 inputs up to 16 batch rows, 2048 above)
    for (N, K, kp), nt in itertools.product([(16, 128, 4096), (1, 128, 4096), (33, 384, 4096), (37, 1152, 4096),
                                             (95, 2176, 2048), (96, 2176, 2048), (100, 4224, 4096), (61, 11008, 2048)],
                                            range(1, 7)):
        tiles = (N + 15) // 16
        for t0 in range(tiles):
            if t0 + nt > tiles:
                continue
            seen = (ctypes.c_ubyte * (N * K * bits // 128 + 1))()
            missing = ctypes.c_long()
            bad = walk(N, K, bits, t0 * 16, nt, kp, seen, ctypes.byref(missing))
            assert (bad, missing.value) == (0, 0), (N, K, t0, nt)


def test_the_last_offsets_do_not_wrap(walk):
    # the longest rows and runs the kernel takes: 6 tiles and two requests ahead of 65536-byte rows
    seen = (ctypes.c_ubyte * (112 * 32768 * 16 // 128 + 1))()
    missing = ctypes.c_long()
    assert walk(112, 32768, 16, 16, 6, 2048, seen, ctypes.byref(missing)) == 0 and missing.value == 0


MIXES = [[(14848, 5120, 16), (12741, 512, 4), (1408, 5120, 8), (21248, 5120, 4)],
         [(15360, 28288, 8), (5632, 512, 4), (9856, 11008, 8)],
         [(5376, 8192, 4), (512, 8192, 4), (2304, 8192, 4), (14514, 8192, 4), (1379, 5248, 4), (23158, 8192, 4),
          (11155, 768, 4), (14720, 8192, 4)],
         [(4096, 4096, 8), (4096, 4096, 4), (4096, 4096, 8)], [(1, 128, 4)], [(11008, 4096, 16), (17, 32768, 4)],
         [(98304, 32768, 16)]]


@pytest.mark.parametrize("blocks", [1, 2])
@pytest.mark.parametrize("mix", MIXES)
def test_division_of_a_launch(lib, mix, blocks):
    count = len(mix)
    tiles = [(n + 15) // 16 for n, _, _ in mix]
    shares = min(256, sum(tiles))
    arr = [(ctypes.c_int * count)(*[m[j] for m in mix]) for j in range(3)]
    out = (ctypes.c_int * (2 * shares * count))()
    lib.divide(count, *arr, blocks, shares, out)
    most = 0
    for e in range(count):
        ranges = [(out[2 * (i * count + e)], out[2 * (i * count + e) + 1]) for i in range(shares)]
        assert ranges[0][0] == 0 and ranges[-1][1] == tiles[e]
        assert all(a <= b for a, b in ranges) and all(x[1] == y[0] for x, y in zip(ranges, ranges[1:]))
        most = max(most, max(b - a for a, b in ranges))
    # A tile takes half a microsecond however short its rows are, and the launch at least as long as its weights do at
    # 6.5 TB/s: no workgroup may get so many short tiles that the launch waits for it.
    stream_us = sum(n * k * b / 8 for n, k, b in mix) / 6.5e6
    assert 0.5 * most <= 2 * stream_us + 2


@pytest.mark.parametrize("blocks,panel,turn,wait", [(1, 4096, 11, 55), (2, 2048, 25, 30)])
def test_a_tile_costs_what_was_fitted_for_its_batch_rows(lib, blocks, panel, turn, wait):
    # The kernel hands the cost its number of 16-row blocks and nothing else.  Up to 16 batch rows a panel of x is 4096 inputs
    # and its figures are the first ones, above 2048 and the second: the fit written out.
    assert lib.panel_of(blocks) == panel
    for bits, fixed, per_group in ((4, 66, 5.4), (8, 66, 7.5), (16, 40, 14.2)):
        for K in list(range(128, 4352, 128)) + [5120, 8192, 11008, 28672, 32768]:
            turns = sum(-(-min(panel, K - k) * bits // 8192) for k in range(0, K, panel))   # 8 lines of 128 bytes each
            want = fixed + int(K // 128 * per_group + 1e-6) + turns * turn + (-(-K // panel) - 1) * wait
            assert lib.tile_cost(blocks, K, bits) == want, (bits, K)
