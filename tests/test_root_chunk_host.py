"""How many root items of a plan a wavefront takes at a time: two, whose queue updates cost half,
unless wavefronts would be left without an item."""
import pytest

from emu import emu


# resident wavefronts 4096; the items of the plans that were measured by ones and by twos
@pytest.mark.parametrize("items, chunk", [(0, 1), (236, 1), (3850, 1), (5448, 1), (7496, 2), (9587, 2), (13126, 2),
                                          (24826, 2), (26341, 2), (98375, 2)])
def test_measured_plans(items, chunk):
    assert emu.root_chunk(items, 4096) == chunk


def test_no_wavefront_is_left_without_half_of_its_share():
    for items in range(0, 20000, 7):
        c = emu.root_chunk(items, 4096)
        assert c == 1 or (items + c - 1) // c >= 4096 * 3 // 4
