"""Which stages of a stage-ordered plan go without a grid barrier (csrc/fq_staged_src.h, compiled for the host here),
against the rule written out over every pair of entries, on random plans with chained, shared, shifted, reused and
overlapping buffers (CPU only)."""
import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_12024_amd", "csrc")
DRIVER = r"""
#include "fq_staged_src.h"
extern "C" void sources(int count, const uintptr_t *x, const uintptr_t *y, const int *K, const int *N, const int *stage,
                        const int *begin, int n_stages, int *src)
{
    staged_sources(count, x, y, K, N, stage, begin, n_stages, src);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("src")
    (d / "t.cpp").write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t.so")])
    return ctypes.CDLL(str(d / "t.so"))


def _run(lib, xs, ys, Ks, Ns, stage):
    n = len(xs)
    begin = [i for i in range(n) if i == 0 or stage[i] != stage[i - 1]] + [n]
    src = (ctypes.c_int * n)()
    lib.sources(n, (ctypes.c_size_t * n)(*xs), (ctypes.c_size_t * n)(*ys), (ctypes.c_int * n)(*Ks), (ctypes.c_int * n)(*Ns),
                (ctypes.c_int * n)(*stage), (ctypes.c_int * len(begin))(*begin), len(begin) - 1, src)
    return list(src)


def _rule(xs, ys, Ks, Ns, stage):
    n = len(xs)
    meets = lambda a, la, b, lb: a < b + 2 * lb and b < a + 2 * la
    inside = [[y <= x and x + 2 * K <= y + 2 * N for y, N in zip(ys, Ns)] for x, K in zip(xs, Ks)]
    for a in range(n):
        for b in range(n):
            if a < b and meets(ys[a], Ns[a], ys[b], Ns[b]):
                return [0] * n
            if meets(xs[a], Ks[a], ys[b], Ns[b]) and not (inside[a][b] and stage[b] < stage[a]):
                return [0] * n
    src = [0] * n
    for s in range(2, max(stage) + 1):
        own = [e for e in range(n) if stage[e] == s]
        of = [next((b + 1 for b in range(n) if inside[e][b] and stage[b] == s - 1), 0) for e in own]
        if all(of):
            for e, v in zip(own, of):
                src[e] = v
    return src


@pytest.mark.parametrize("seed", range(8))
def test_the_rule_over_random_plans(lib, seed):
    rng = random.Random(seed)
    polled = refused = 0
    for _ in range(400):
        n = rng.randint(1, 12)
        stage = [0]
        for _ in range(n - 1):
            stage.append(stage[-1] + rng.randint(0, 1))
        Ks = [128 * rng.randint(1, 4) for _ in range(n)]
        Ns = [rng.choice([128, 256, 512, 500, 130]) for _ in range(n)]
        odd = rng.random() < 0.5      # a plan with a buffer used in some way of its own
        xs, ys, top = [], [], 4096
        for i in range(n):
            earlier = [b for b in range(i) if stage[b] == stage[i] - 1 and Ns[b] >= Ks[i]]
            if earlier and rng.random() < 0.9:
                b = rng.choice(earlier)
                xs.append(ys[b] + 16 * rng.randint(0, (Ns[b] - Ks[i]) // 8))
            else:
                xs.append(top)
                top += 2 * Ks[i] + 16
            ys.append(top)
            top += 2 * Ns[i] + 16 * rng.randint(0, 1)
            if odd and rng.random() < 0.1:
                ys[-1] = rng.choice(ys) + 2 * rng.randint(0, 300)
            if odd and rng.random() < 0.1:
                xs[-1] = rng.choice(xs + ys) + 16 * rng.randint(0, 40)
        want = _rule(xs, ys, Ks, Ns, stage)
        assert _run(lib, xs, ys, Ks, Ns, stage) == want, (xs, ys, Ks, Ns, stage)
        polled += any(want)
        refused += not any(want) and max(stage) > 1
    assert polled > 40 and refused > 40
