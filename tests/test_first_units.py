"""Every unit of a persistent launch is taken once, whatever the number of CUs: blocks begin with units by their numbers, counters deal out the rest.  A unit that
waits for others does so inside its own queue."""
import heapq
import itertools

import numpy as np
import pytest

from host_rules import deals_first, first_unit, head_queues, keeps_reserve, persistent_blocks, unit_numbers

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


def _makespan(units, blocks, held, deal, reserve):
    """When a launch ends whose units, longest first, are taken as the kernels take them, and `held` of whose blocks can only begin when another has run dry.
    deal: blocks begin by number.  reserve: a block has its next unit from the unit before."""
    n = len(units)
    counter = itertools.count(blocks if deal else 0)
    late = list(range(blocks - held, blocks))
    events, ahead, end = [(0., b) for b in range(blocks - held)], {}, 0.
    while events:
        t, b = heapq.heappop(events)
        if b not in ahead:                                   # it begins
            unit = b if deal else next(counter)
        else:
            unit = ahead[b] if reserve else next(counter)
        ahead[b] = next(counter) if reserve else -1
        if unit < n:
            end = t + units[unit]
            heapq.heappush(events, (end, b))
        elif late:
            heapq.heappush(events, (t, late.pop(0)))
    return max(end, t)


def _rule(n, blocks, per_block, longest):
    deal = deals_first(n, blocks, per_block, longest)
    return deal, keeps_reserve(deal, longest)


@pytest.mark.parametrize("n,blocks,held", [(600, 32, 2), (300, 64, 4), (2000, 96, 6)])
def test_blocks_that_cannot_start_hold_no_long_unit_back(n, blocks, held):
    """A launch of many units ends within the length of the last units of the least time on the blocks that can start (a block that runs dry begins no unit
    after the others' last ones).  With first units by number it ends with a unit of the longest."""
    units = [100. - 99. * i / n for i in range(n)]
    least = sum(units) / (blocks - held)
    by_number = _makespan(units, blocks, held, True, True)
    assert _makespan(units, blocks, held, *_rule(n, blocks, 4, 4096)) <= min(least + units[n - blocks], by_number - 0.4 * units[0])
    assert by_number >= least + 0.5 * units[0]


@pytest.mark.parametrize("per_block", [4, 32])
@pytest.mark.parametrize("longest", [0, 64, 1024, 1025, 65536])
def test_when_blocks_begin_by_number(per_block, longest):
    most = (per_block if longest <= 1024 else 2) * 96
    assert deals_first(most, 96, per_block, longest) and not deals_first(most + 1, 96, per_block, longest) and not deals_first(1, 0, per_block, longest)
    assert keeps_reserve(True, longest) == (longest <= 1024) and not keeps_reserve(False, longest)


@pytest.mark.parametrize("n,blocks", [(648, 256), (1128, 768), (300, 256)])
def test_long_units_end_evenly(n, blocks):
    """Units of a long sequence, one to two and a half per block: list scheduling, as no block has a unit that another could begin, which ends within a
    longest unit of the mean load (the unit that ends last began when no block was free before)."""
    units = [min(331., 331. * (n - i) / 300) for i in range(n)]
    deal, reserve = _rule(n, blocks, 32, 40000)
    assert not reserve and _makespan(units, blocks, 0, deal, reserve) <= sum(units) / blocks + units[0]


def test_units_in_reserve_make_the_end_uneven():
    """Why: 648 units of a sharded sequence on 256 blocks."""
    units = [min(331., 331. * (648 - i) / 300) for i in range(648)]
    assert _makespan(units, 256, 0, False, False) <= 1.1 * sum(units) / 256 < _makespan(units, 256, 0, False, True)


def test_grids():
    assert persistent_blocks(256, 10 ** 9) == 256 and persistent_blocks(768, 767) == 768 and persistent_blocks(768, 41) == 48
    assert persistent_blocks(300, 10 ** 9) == 296 and persistent_blocks(4, 10) == 8 and persistent_blocks(256, 0) == 8


def _list(block, per_tile, in_turn, n_tiles):
    """The (tile, head) units that the block's counter deals out, in that order, and the counter."""
    queues = head_queues(per_tile, in_turn)
    here = per_tile // queues
    assert here * queues == per_tile
    counter, mul, add = unit_numbers(block, queues, in_turn)
    return counter, [(u // here, block % queues * here + u % here) for u in range(add, n_tiles * here, mul)]


@pytest.mark.parametrize("in_turn", [0, 1])
@pytest.mark.parametrize("per_tile", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 15, 20, 24, 11, 13, 40, 64])
def test_queues_cover_every_unit_and_pieces_wait_in_their_own(per_tile, in_turn):
    n_tiles = 37
    queue = {}                                               # counter -> its units
    for block in range(24):                                  # (the first eight have a block in every queue)
        counter, units = _list(block, per_tile, in_turn, n_tiles)
        assert 0 <= counter < XCDS and queue.setdefault(counter, units) == units
    assert sorted(u for units in queue.values() for u in units) == [(t, h) for t in range(n_tiles) for h in range(per_tile)]
    for counter, units in queue.items():
        assert units == sorted(units)                        # list order
        if in_turn:                                          # a head's tiles, pieces among them, are all here
            heads = {h for _, h in units}
            assert len(units) == n_tiles * len(heads)
            assert len(heads) * head_queues(per_tile, 1) == per_tile
    assert {_list(b, per_tile, in_turn, n_tiles)[0] for b in range(XCDS)} == set(queue)
