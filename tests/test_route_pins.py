"""Host-side choices of the launch code that need no device (CPU only)."""
from plan_util import part_mutex


def test_calls_on_different_streams_and_devices_share_no_lock():
    # the lock that keeps the two launches of a product split along K together belongs to one array of partial sums
    locks = [part_mutex(d, b) for d in (0, 1, 63) for b in range(4)]
    assert None not in locks and len(set(locks)) == len(locks)
    assert part_mutex(0, 2) == locks[2]
