"""The forward's tile list fits the memory it is built in: a caller's scratch buffer, and the 2 MiB of fcp_attn_fwd_step_static."""
import numpy as np
import pytest

from paper_2602_21788_amd import binding as B

from host_rules import forward_plan, lib

STATIC = 2 * 1024 * 1024
HEADS = [(1, 1), (2, 1), (4, 4), (6, 2), (8, 1), (8, 2), (10, 2), (32, 8), (40, 8), (64, 8)]


def _most_tiles(tq, tkv, n_work, n_parts, tile):
    """Tiles of a list that covers every row in every partial slot, as far as there are keys for that."""
    return n_work + min(n_parts * -(-tq // tile), -(-tkv // tile))


def _region(n_work, tiles):
    """Header, item offsets and 64-byte tile records."""
    return -(-(128 + -(-(n_work + 1) * 4 // 64) * 64 + tiles * 64) // 256) * 256


@pytest.mark.parametrize("head_dim,hq,hkv,tq,tkv,n_parts", [
    (64, 2, 1, 697_500, 2_790_000, 4),      # 64-row tiles: 0.7 MB past the end
    (64, 2, 1, 418_750, 3_350_000, 8),
    (64, 4, 2, 525_000, 2_100_000, 4),
    (128, 2, 1, 525_000, 2_100_000, 4),     # (many short items)
])
def test_static_area_just_below_its_limit(head_dim, hq, hkv, tq, tkv, n_parts):
    n_work = 4 * n_parts if head_dim == 64 else 4200
    assert lib().static_bytes(tq, tkv, n_work, n_parts) <= STATIC          # accepted
    tile, pair, cap, region = forward_plan(head_dim, hq, hkv, tq, tkv, n_work, n_parts, STATIC)
    assert cap >= _most_tiles(tq, tkv, n_work, n_parts, tile) and _region(n_work, cap) == region <= STATIC
    assert forward_plan(head_dim, hq, hkv, tq, tkv, n_work, n_parts, 1 << 40)[3] > STATIC      # what an unlimited area would be given


def test_every_list_fits_its_area():
    rng = np.random.default_rng(5)
    near = 0
    for _ in range(20000):
        hq, hkv = HEADS[rng.integers(len(HEADS))]
        head_dim, n_parts = int(rng.choice([64, 128])), int(rng.integers(1, 9))
        if rng.integers(2):                                   # 2 to 4 M pool keys: about what the static area takes
            tkv = int(rng.integers(2_000_000, 4_000_000))
            tq = int(tkv * rng.uniform(0.5, 1.1) / n_parts) + 1
        else:
            tkv = int(np.exp(rng.uniform(0, np.log(4e6)))) + 1
            tq = int(rng.integers(0, tkv + 1))
        n_work = int(np.exp(rng.uniform(0, np.log(30000))))
        n_cu = int(rng.choice([32, 100, 256, 304]))
        for area in (STATIC, lib().scratch_area_bytes(tq, tkv, n_work, n_parts)):
            if area == STATIC and lib().static_bytes(tq, tkv, n_work, n_parts) > STATIC:
                continue                                      # refused
            tile, pair, cap, region = forward_plan(head_dim, hq, hkv, tq, tkv, n_work, n_parts, area, n_cu)
            what = (head_dim, hq, hkv, tq, tkv, n_work, n_parts, n_cu, area)
            assert tile in (32, 64, 128, 256) and cap >= _most_tiles(tq, tkv, n_work, n_parts, tile), what
            assert _region(n_work, cap) <= area, what
            assert not pair or (hq // hkv) % 2 == 0, what
            near += forward_plan(head_dim, hq, hkv, tq, tkv, n_work, n_parts, 1 << 40, n_cu)[3] > area
    assert near > 100                                         # the limit was met


def test_a_scratch_buffer_has_room_for_the_smallest_tiles():
    """The work area beside the row states (a byte per row), and a buffer for the largest call has room for smaller ones."""
    rng = np.random.default_rng(6)
    for _ in range(400):
        big = [int(rng.integers(1, 70000)), int(rng.integers(1, 70000)), int(rng.integers(1, 3000)), int(rng.integers(1, 9))]
        small = [int(rng.integers(1, x + 1)) if rng.integers(0, 3) else x for x in big]
        size = [B.fcp_scratch_bytes(B.FCP_SCRATCH_FWD, tq, tkv, 8, 2, 128, n, parts) for tq, tkv, n, parts in (big, small)]
        assert size[1] <= size[0], (big, small)
        tq, tkv, n, parts = big
        assert size[0] >= _region(n, _most_tiles(tq, tkv, n, parts, 32)) + tq, big
