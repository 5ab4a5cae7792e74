"""Every eigenvalue of a small single problem is asked for by a thread of its own, also on a device
that reports few compute units (or none: the library then counts one)."""
import pytest

from emu import emu

BLOCK, FIN_MAX = 256, 1280


@pytest.mark.parametrize("cus", [1, 2, 4, 5, 20, 256, 304])
def test_a_thread_per_eigenvalue(cus):
    for n in range(1, FIN_MAX + 1):
        blocks = emu.finish_redo_blocks(n, cus, BLOCK)
        assert 1 <= blocks <= n
        assert (n + blocks - 1) // blocks <= BLOCK   # the first block's share, the largest
        if n <= 3 * cus:
            assert blocks == n                       # no listed eigenvalue waits for another
