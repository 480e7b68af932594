"""Every unit of a persistent launch is taken once, whatever the number of CUs: blocks begin with units by their numbers, counters deal out the rest."""
import numpy as np
import pytest

from host_rules import first_unit, persistent_blocks

XCDS = 8


def _taken(grid, key_units, row_units, n_long):
    """(key, row) units as the blocks of one queue and its counters take them, two lists of that many units; the queue is number 0 of eight."""
    places = grid // XCDS
    keys, rows, dealt = [], [], 0
    for block in range(0, grid, XCDS):                       # the queue's blocks
        dealt, key, row = first_unit(block // XCDS, places, key_units, min(n_long, key_units, places))
        assert (key >= 0) != (row >= 0)
        keys += [key] if 0 <= key < key_units else []
        rows += [row] if 0 <= row < row_units else []
    keys += range(dealt, key_units)
    rows += range(places - dealt, row_units)
    return sorted(keys), sorted(rows)


@pytest.mark.parametrize("n_cu", [1, 7, 8, 20, 32, 38, 76, 100, 228, 256, 304])
def test_every_unit_once(n_cu):
    rng = np.random.default_rng(n_cu)
    for per_cu in (1, 2, 3):
        for _ in range(60):
            key_units, row_units = (int(np.exp(rng.uniform(0, 8))) - 1 for _ in range(2))
            grid = persistent_blocks(n_cu * per_cu, XCDS * (key_units + row_units))
            assert grid % XCDS == 0 and XCDS <= grid <= max(XCDS, n_cu * per_cu)
            keys, rows = _taken(grid, key_units, row_units, int(rng.integers(0, 1 + grid // XCDS)))
            assert keys == list(range(key_units)) and rows == list(range(row_units)), (grid, key_units, row_units)


def test_a_grid_that_is_no_multiple_takes_units_twice():
    """Why: 300 blocks, a 38th block in queues 0 to 3."""
    keys, rows = _taken(300, 200, 200, 0)
    assert len(rows) > len(set(rows))


def test_grids():
    assert persistent_blocks(256, 10 ** 9) == 256 and persistent_blocks(768, 767) == 768 and persistent_blocks(768, 41) == 48
    assert persistent_blocks(300, 10 ** 9) == 296 and persistent_blocks(4, 10) == 8 and persistent_blocks(256, 0) == 8
