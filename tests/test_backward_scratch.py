"""The backward's scratch buffer has room for everything that its lists can hold."""
import numpy as np

import pytest

from host_rules import backward_caps
from paper_2602_21788_amd import binding as B


def _list_capacity(tkv, n_work):
    """Key tiles that the backward's list has room for."""
    return 2 * (2 * n_work + 2 * -(-tkv // 128)) + 2048


def test_chain_records_for_every_tile_of_a_full_list():
    """With 128 channels per head the scratch holds, beside the areas of any backward, a 16-byte chain record per key tile and a flag word
    per (32-row block, head, eighth of the block)."""
    rng = np.random.default_rng(1)
    for _ in range(300):
        hkv = int(rng.choice([1, 2, 8, 16]))
        hq = hkv * int(rng.integers(1, 5))
        tq, n_work = int(rng.integers(1, 40000)), int(rng.integers(1, 1025))
        tkv = tq + int(rng.integers(0, 2)) * int(rng.integers(0, 40000))
        size = [B.fcp_scratch_bytes(B.FCP_SCRATCH_BWD, tq, tkv, hq, hkv, D, n_work, 1) for D in (64, 128)]
        flags = (tq // 32 + 1 + n_work) * hq * 8 * 4
        if hkv % 8 == 0:
            assert size[1] - size[0] >= _list_capacity(tkv, n_work) * 16 + flags, (tq, tkv, hq, hkv, n_work)
        else:                                                 # the one-pass backward does not take such heads
            assert size[1] == size[0], (tq, tkv, hq, hkv, n_work)


def test_a_buffer_for_the_largest_call_has_room_for_smaller_ones():
    """Programs size the scratch once: a call with fewer rows, keys or items of the same heads never needs more."""
    rng = np.random.default_rng(2)
    for _ in range(400):
        hkv = int(rng.choice([1, 2, 3, 8, 16]))
        hq, D = hkv * int(rng.integers(1, 5)), int(rng.choice([64, 128]))
        big = [int(rng.integers(1, 70000)), int(rng.integers(1, 70000)), int(rng.integers(1, 3000))]
        small = [int(rng.integers(1, x + 1)) if rng.integers(0, 3) else x for x in big]
        size = [B.fcp_scratch_bytes(B.FCP_SCRATCH_BWD, tq, tkv, hq, hkv, D, n_work, 1) for tq, tkv, n_work in (big, small)]
        assert size[1] <= size[0], (big, small, hq, hkv, D)


def _up(a, b):
    return -(-a // b)


def _pieces(items, group, hkv, pair, n_cu):
    """(key tiles, query tiles) with their pieces, counted as the scheduler does for causal items (rows, first row, keys): the size of a piece is a CU's share
    of the steps, counted from the first and last tile of each item, and no less than 12 steps.  (Its other lower bounds make fewer pieces.)"""
    bm = 64 if pair else 128
    c = lambda n, lo, k: _up(n - min(n - 1, max(0, k - lo)), 32)          # 32-row blocks of the item that see key k
    keys = rows = 0.
    for n, lo, kv in items:
        nt, nq = _up(kv, 128), _up(n, bm)
        keys += 0.5 * nt * (c(n, lo, 0) + c(n, lo, (nt - 1) * 128)) * group * hkv
        rows += 0.25 * nq * (_up(min(lo + min(n, bm), kv), 32) + _up(kv, 32)) * (group * hkv // (2 if pair else 1))
    cut_rows = 32 * max(1, int(max(keys / n_cu, 12)) // group)
    cut_keys = 32 * int(max(rows / n_cu, 12))
    return (sum(_up(kv, 128) * _up(n, cut_rows) for n, lo, kv in items), sum(_up(n, bm) * max(1, _up(kv, cut_keys)) for n, lo, kv in items))


@pytest.mark.parametrize("pair", [False, True])
def test_lists_have_room_for_every_piece(pair):
    """Every size of a piece that the scheduler can choose leaves both lists below their capacity: a tile beyond it would be dropped.  The number of query
    tiles beyond two per tile comes close to the most that the bound allows (four per CU and a little), so that a cut half as fine again would be seen."""
    rng = np.random.default_rng(3)
    most = [0, 0]
    for i in range(3000):
        n_cu, hkv = int(rng.choice([64, 256, 304, 470])), int(rng.choice([1, 1, 2, 3, 8]))
        group = int(rng.choice([2, 4, 14])) if pair else int(rng.choice([1, 3, 5]))
        n_work = int(rng.choice([1, 1, 2, 30, 1024]))
        length = np.exp(rng.uniform(0, np.log(200000. / n_work), n_work)).astype(int) + 1
        lo = rng.integers(0, 4, n_work) * rng.integers(0, 1 + 100000 // n_work)         # rows of earlier ranks
        items = [(int(n), int(a), int(n + a)) for n, a in zip(length, lo)]
        tq, tkv = sum(n for n, _, _ in items), sum(kv for _, _, kv in items)
        for j, (have, cap) in enumerate(zip(_pieces(items, group, hkv, pair, n_cu), backward_caps(tq, tkv, n_work))):
            assert have <= cap, (items[:4], group, hkv, n_cu)
            tiles = sum(_up(kv, 128) if j == 0 else _up(n, 64 if pair else 128) for n, _, kv in items)
            most[j] = max(most[j], (have - 2 * tiles) / n_cu)
    assert most[0] <= 4 and most[1] <= 4 * 13 / 12 and most[1] >= 3, most
