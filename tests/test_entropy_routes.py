"""How the entropies' rows are taken (fq_entropy_route, a host function): what the kernels and their scratch assume of it (CPU only)."""
import random

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
