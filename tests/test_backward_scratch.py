"""The backward's scratch buffer has room for everything that its lists can hold."""
import numpy as np

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
