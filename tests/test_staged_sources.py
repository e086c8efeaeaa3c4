"""Which stages of a stage-ordered plan go without a grid barrier (csrc/fq_staged_src.h, compiled for the host here),
against the rule written out over every pair of entries, on random plans with chained, shared, shifted, reused and
overlapping buffers; and that nobody waits for rows of a share that is refused: the deal of the kernel written out, over
the widths that the entries may be switched to (CPU only)."""
import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_12024_amd", "csrc")
DRIVER = r"""
#include "fq_staged_src.h"
extern "C" void sources(int count, const uintptr_t *x, const uintptr_t *y, const int *K, const int *N, const int *widths,
                        const int *stage, const int *begin, int n_stages, int grid, int most, int *src)
{
    staged_sources(count, x, y, K, N, widths, stage, begin, n_stages, grid, most, src);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("src")
    (d / "t.cpp").write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t.so")])
    return ctypes.CDLL(str(d / "t.so"))


def _run(lib, xs, ys, Ks, Ns, stage, widths=None, grid=256, most=1024):
    n = len(xs)
    begin = [i for i in range(n) if i == 0 or stage[i] != stage[i - 1]] + [n]
    src = (ctypes.c_int * n)()
    lib.sources(n, (ctypes.c_size_t * n)(*xs), (ctypes.c_size_t * n)(*ys), (ctypes.c_int * n)(*Ks), (ctypes.c_int * n)(*Ns),
                (ctypes.c_int * n)(*(widths or [31] * n)), (ctypes.c_int * n)(*stage), (ctypes.c_int * len(begin))(*begin),
                len(begin) - 1, grid, most, src)
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


COST = {2: 64 * 230 * 730 // 1000, 3: 64 * 230 * 950 // 1000, 4: 64 * 230, 8: 128 * 200, 16: 256 * 200}


def _largest_shares(Ks, Ns, bits, grid):
    """Chunks of 4 rows in the largest share of each entry of one stage, dealt as the kernel deals (0 bits: not run)."""
    cost = [COST.get(b, 0) * (K >> 7) * ((N + 3) >> 2) for K, N, b in zip(Ks, Ns, bits)]
    left, out, prefix = grid - len(Ks), [], 0
    for e, (N, c) in enumerate(zip(Ns, cost)):
        lo = e + left * prefix // max(sum(cost), 1)
        prefix += c
        n = e + 1 + left * prefix // max(sum(cost), 1) - lo
        chunks = (N + 3) >> 2
        out.append(max(chunks * (i + 1) // n - chunks * i // n for i in range(n)) if c else 0)
    return out


def _staircase(Ns, Ks, readers):
    """Stage 0, one linear; stage 1 of the given linears, each with an x of its own; stage 2 whose entries read their ys."""
    xs, ys, KK, NN, stage, top = [1 << 20], [2 << 20], [128], [128], [0], 4 << 20
    for N, K in zip(Ns, Ks):
        xs.append(top), ys.append(top + 2 * K), KK.append(K), NN.append(N), stage.append(1)
        top += 2 * K + 2 * N + 64 & ~15
    for r in readers:
        xs.append(ys[1 + r]), ys.append(top), KK.append(128), NN.append(128), stage.append(2)
        top += 512
    return xs, ys, KK, NN, stage


def test_rows_that_no_workgroup_may_hold_are_not_waited_for(lib):
    # 40000 short rows beside 1500 of 32768 inputs: at 4 and 16 bits the short ones are dealt 9 of 256 workgroups, 1112 chunks each
    for Ks, bits, waits in ([128, 32768], (4, 16), 0), ([4096, 32768], (4, 16), 1), ([128, 4096], (4, 16), 1):
        plan = _staircase([40000, 1500], Ks, [0])
        got = _run(lib, *plan[:4], plan[4], [31, 1 << 2, 1 << 4, 31])
        assert got == [0, 0, 0, 2 * waits], Ks
        assert (max(_largest_shares(Ks, [40000, 1500], bits, 256)) > 1024) == (not waits)


@pytest.mark.parametrize("seed", range(4))
def test_no_share_that_is_waited_for_is_refused(lib, seed):
    rng = random.Random(seed)
    waited = kept_back = refused = 0
    for _ in range(300):
        n, grid, most = rng.randint(1, 6), rng.choice([8, 64, 256]), rng.choice([4, 32, 1024])
        Ks = [128 * rng.choice([1, 2, 8, 32, 86, 256]) for _ in range(n)]
        Ns = [max(128, int(min(400, most) * grid * 4 * rng.random() ** 4)) for _ in range(n)]
        sets = [rng.sample(sorted(COST), rng.randint(1, 5)) for _ in range(n)]
        plan = _staircase(Ns, Ks, range(n))
        widths = [31] + [sum(1 << sorted(COST).index(b) for b in s) for s in sets] + [31] * n
        src = _run(lib, *plan[:4], plan[4], widths, grid, most)[1 + n:]
        assert src in ([0] * n, list(range(2, n + 2)))
        most_seen = 0
        for _ in range(60):
            bits = [rng.choice(s + [0]) if rng.random() < 0.1 else rng.choice([min(s), max(s)]) for s in sets]
            most_seen = max(most_seen, *_largest_shares(Ks, Ns, bits, grid))
        assert not any(src) or most_seen <= most, (Ks, Ns, sets, grid, most)
        waited += any(src)
        kept_back += not any(src)
        refused += most_seen > most
    assert waited > 30 and refused > 30 and kept_back < refused + 40     # (the rule looks at no more widths than there are)
