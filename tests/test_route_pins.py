"""Host-side choices of the launch code that need no device (CPU only)."""
import pytest

from plan_util import batch_serves, batch_serves_linear, batch_serves_narrow, batch_serves_slab, part_mutex, prompt_plan, w8a8_plan


def test_calls_on_different_streams_and_devices_share_no_lock():
    # the lock that keeps the two launches of a product split along K together belongs to one array of partial sums
    locks = [part_mutex(d, b) for d in (0, 1, 63) for b in range(4)]
    assert None not in locks and len(set(locks)) == len(locks)
    assert part_mutex(0, 2) == locks[2]


@pytest.mark.parametrize("N,K,bits,M,batch", [
    (4096, 4096, 4, 16, True), (11008, 4096, 8, 32, True), (28672, 8192, 4, 16, True), (12288, 128, 4, 2, True),
    # short rows over many tiles; many rows; tiles of the register-fed kernel that fill their rounds
    (32768, 512, 4, 16, False), (55552, 512, 4, 24, False), (65536, 1024, 8, 2, False), (40960, 512, 16, 17, False),
    (128256, 4096, 4, 16, True), (131071, 8192, 8, 32, True), (131072, 8192, 8, 32, False), (32768, 5120, 4, 16, False), (30720, 3072, 4, 32, False),
    (32768, 4096, 4, 16, True), (32768, 4096, 4, 17, False), (28672, 8192, 4, 32, True), (28672, 3072, 4, 32, False)])
def test_single_calls_take_the_faster_small_batch_kernel(N, K, bits, M, batch):
    # (a host without a device counts 256 compute units)
    assert batch_serves_linear(N, K, bits, M) is batch


STACKS = {"7b": (4096, 11008, 4096), "13b": (5120, 13824, 5120), "70b": (8192, 28672, 1024)}


@pytest.mark.parametrize("widths", [(4,), (8,), (4, 8), (4, 8, 16)])
@pytest.mark.parametrize("M", [2, 16])
@pytest.mark.parametrize("stack", list(STACKS))
def test_stages_of_a_decoder_run_on_the_small_batch_kernel(stack, M, widths):
    h, ffn, kv = STACKS[stack]
    for stage in ([(h, h), (kv, h), (kv, h)], [(h, h)], [(ffn, h)] * 2, [(h, ffn)]):
        assert batch_serves([(N, K, widths) for N, K in stage], M), stage


@pytest.mark.parametrize("entries,M,batch", [
    ([(16384, 512, (4, 8))] * 4, 2, False), ([(24576, 1024, (4,))] * 3, 16, False),   # short rows
    ([(1024, 512, (4, 8))] * 8, 2, True),                                             # two tiles per compute unit
    ([(16384, 5120, (4,))] * 4, 16, False), ([(16384, 4096, (4,))] * 4, 16, True),    # full rounds of the other kernel
    ([(16384, 4096, (4,))] * 4, 17, False), ([(16384, 4096, (4, 8))] * 4, 17, True),
    ([(8192, 4096, (4, 8))] * 13, 16, False), ([(16, 4096, (4, 8))] * 65, 16, False)])  # rows and entries of a plan
def test_plans_take_the_faster_small_batch_kernel(entries, M, batch):
    assert batch_serves(entries, M) is batch


@pytest.mark.parametrize("widths", [(2,), (3,), (2, 4, 8), (3, 4, 8)])
@pytest.mark.parametrize("M", [2, 16, 17, 32])
@pytest.mark.parametrize("stack", list(STACKS))
def test_stages_with_narrow_copies_run_on_the_small_batch_kernel(stack, M, widths):
    h, ffn, kv = STACKS[stack]
    for stage in ([(h, h), (kv, h), (kv, h)], [(h, h)], [(ffn, h)] * 2, [(h, ffn)]):
        # (two part panels of x: a narrow copy alone over more than two tiles per compute unit stays)
        stays = h == 5120 and len(stage) > 1 and len(widths) == 1 and M <= 16
        assert batch_serves([(N, K, widths) for N, K in stage], M) is not stays, stage


W2, W3 = (2, 4, 8), (3, 4, 8)


@pytest.mark.parametrize("entries,M,own_x,batch", [
    ([(16384, 512, (2,))] * 4, 2, False, False), ([(12289, 2048, (3,))], 17, False, False), ([(12289, 4096, (3,))], 17, False, True),
    ([(30000, 3072, W2)] * 3, 2, False, True), ([(30000, 3072, (2,))] * 3, 2, False, False),            # short rows
    ([(8192, 8192, (3,))] * 12, 16, True, True), ([(8192, 8192, (3,))] * 13, 16, True, False),          # rows of a plan
    ([(6000, 5120, W2)] * 3, 16, True, True), ([(6000, 5120, W2)] * 5, 16, True, False),                # part panels, full rounds
    ([(6000, 5120, W2)] * 5, 17, True, True), ([(6000, 5120, W3)] * 8, 2, False, False), ([(6000, 5120, (4, 8))] * 5, 16, True, True),
    ([(30000, 5120, W2)], 16, False, True), ([(2048, 6144, W2)] * 24, 16, True, False), ([(512, 6144, W2)] * 60, 16, True, True),
    ([(1000, 8192, W3)] * 30, 17, True, False), ([(1000, 8192, W3)] * 30, 17, False, True),             # short entries, an x each
    ([(1000, 8192, W3)] * 30, 16, True, True), ([(1000, 8192, W3)] * 50, 32, True, True), ([(1200, 11008, W3)] * 24, 32, True, True),
    ([(512, 6144, W3)] * 60, 32, True, True), ([(1000, 8192, (4, 8))] * 30, 32, True, True)])
def test_plans_with_narrow_copies_take_the_faster_small_batch_kernel(entries, M, own_x, batch):
    assert batch_serves(entries, M, own_x) is batch


@pytest.mark.parametrize("bits", [2, 3])
@pytest.mark.parametrize("N,K,M,batch", [(4096, 4096, 16, True), (8192, 128, 2, True), (8193, 1152, 20, False), (8193, 4096, 32, True), (8193, 5120, 16, False),
                                         (8193, 5120, 17, True), (98304, 8192, 2, True), (98305, 8192, 2, False)])
def test_single_narrow_calls_take_the_faster_small_batch_kernel(N, K, M, bits, batch):
    assert batch_serves_narrow(N, K, bits, M) is batch


@pytest.mark.parametrize("N,K,M,batch", [(4096, 4096, 32, True), (1000, 896, 2, False), (1000, 1024, 2, True), (16384, 5120, 32, True),
                                         (16385, 5120, 32, False), (16385, 8192, 32, True)])
def test_slabs_of_a_three_bit_prompt(N, K, M, batch):
    assert batch_serves_slab(N, K, M) is batch


@pytest.mark.parametrize("M,N,K,kind,plan", [
    # over few inputs: the large tiles' rounds, no segments of one group each
    (2048, 8192, 128, "group", (0, 0)), (2048, 8192, 640, "group", (0, 0)), (2048, 8192, 1536, "group", (0, 0)),
    (400, 28672, 256, "group", (0, 0)), (33, 512, 512, 16, (2, 1)), (100, 2048, 512, 16, (2, 1)),
    # the shapes the kernels with segments of K were made for
    (100, 4096, 11008, 4, (2, 4)), (515, 11008, 4096, 8, (4, 1)), (300, 5120, 13824, "group", (2, 2)),
    (2048, 28672, 8192, 4, (0, 0)), (2048, 8192, 28672, "row", (0, 0))])
def test_prompts_take_the_faster_tiles(M, N, K, kind, plan):
    got = prompt_plan(M, N, K, kind) if isinstance(kind, int) else w8a8_plan(M, N, K, kind == "row")
    assert got == plan


@pytest.mark.parametrize("M,N,K,kind,large", [
    # a large tile's 256 rows of x or weights are addressed by 32-bit offsets: longer rows go to the smaller tiles
    (2048, 8192, 1 << 23, 4, False), (4096, 65536, 1 << 23, 16, False), (2048, 65536, (1 << 23) - 128, 4, True),
    (2048, 65536, (1 << 23) - 128, 16, True), (4000, 65536, 1 << 24, "group", False),
    (4000, 65536, (1 << 24) - 128, "group", True)])
def test_rows_too_long_for_the_large_tiles(M, N, K, kind, large):
    got = prompt_plan(M, N, K, kind) if isinstance(kind, int) else w8a8_plan(M, N, K, False)
    assert (got == (0, 0)) is large
