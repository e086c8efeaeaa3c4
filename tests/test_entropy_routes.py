"""How the entropies' rows are taken (fq_entropy_route, a host function): what the kernels and their scratch assume of it, and its
two sides at every line (CPU only)."""
import random

import pytest

from plan_util import entropy_route

MAX_PARTS, MAX_PIECES, MAX_SPLIT_ROWS, FINE_ROWS = 2048, 32, 512, 64


def test_pieces_fit_the_scratch_and_one_workgroup():
    rng = random.Random(1)
    sizes = [(R, V) for R in (1, 8, 9, 20, 21, 64, 65, 160, 161, 256, 257, 384, 385, 512, 513)
             for V in (1, 4096, 4097, 6143, 10240, 10241, 65535, 65536, 128256, 2 ** 31 - 1)]
    sizes += [(int(2 ** rng.uniform(0, 11)), int(2 ** rng.uniform(0, 31))) for _ in range(2000)]
    for R, V in sizes:
        for kl in (False, True):
            for half in (False, True):
                for vec in (False, True):
                    for cus in (256, 64, 32):
                        threads, pieces, fine = entropy_route(R, V, kl, half, vec, cus)
                        where = (R, V, kl, half, vec, cus)
                        assert threads in (256, 512) and 1 <= pieces <= MAX_PIECES, where
                        if pieces > 1:  # a piece is a workgroup of 256 threads, the first of a row's pieces is never empty
                            assert threads == 256 and R <= MAX_SPLIT_ROWS and R * pieces <= MAX_PARTS and V >= 1024 * pieces, where
                        if pieces > 1 and R > FINE_ROWS:  # what a workgroup of a whole row can take where the stream has no scratch
                            assert pieces in (4, 8) and not fine, where
                        if R <= FINE_ROWS or (R <= MAX_SPLIT_ROWS and V <= 10240):
                            assert fine, where


@pytest.mark.parametrize("R,V,kl,half,vec,route", [
    (64, 4096, True, False, True, (256, 1, 1)), (512, 4096, True, True, True, (256, 1, 1)), (513, 4096, True, False, True, (256, 1, 0)),
    (64, 4097, True, False, False, (256, 2, 1)), (8, 32000, True, False, True, (256, 31, 1)), (9, 32000, True, False, True, (256, 16, 1)),
    (21, 32000, True, False, True, (256, 8, 1)), (64, 65536, False, True, True, (256, 32, 1)),
    (300, 10240, True, False, True, (256, 1, 1)), (256, 10240, False, False, True, (512, 1, 1)), (257, 10240, False, False, True, (256, 1, 1)),
    (160, 32000, True, False, True, (256, 4, 0)), (161, 32000, True, False, True, (512, 1, 0)), (320, 24575, True, True, True, (256, 4, 0)),
    (321, 24575, True, True, True, (512, 1, 0)), (350, 24576, True, True, True, (256, 4, 0)), (351, 24576, True, True, True, (512, 1, 0)), (160, 65535, True, False, False, (256, 4, 0)), (160, 65536, True, False, True, (256, 8, 0)), (384, 65536, True, False, True, (256, 4, 0)),
    (192, 65536, True, False, True, (256, 8, 0)), (193, 65536, True, False, True, (512, 1, 1)),
    (256, 65536, False, False, True, (256, 8, 0)), (256, 65536, True, True, True, (256, 8, 0)),
    (257, 65536, True, False, True, (256, 4, 0)), (385, 65536, True, False, True, (256, 1, 1)), (385, 90001, True, False, False, (256, 4, 0)),
    (385, 65536, False, False, True, (256, 4, 0)), (512, 65536, True, True, True, (256, 4, 0)), (513, 65536, True, True, True, (512, 1, 0)),
    (1537, 65536, True, True, True, (256, 1, 0)), (513, 65536, True, False, True, (256, 1, 0))])
def test_both_sides_of_the_lines(R, V, kl, half, vec, route):
    assert entropy_route(R, V, kl, half, vec) == route
