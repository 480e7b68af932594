"""Which forward launches do without a list (csrc/fcp_sizes.h): items and slots that a wave holds, and the units it pays for."""
from host_rules import lib

WIDE, SMALL, SPLIT4 = 0, 1, 4


def test_order():
    order = lib().alone_order
    in_list, by_items, by_tiles = 0, 1, 2
    assert order(SMALL, 1, 1280, 256) == in_list and order(SMALL, 2, 256, 256) == in_list
    assert order(SMALL, 2, 257, 256) == by_tiles and order(SPLIT4 - 1, 2, 257, 256) == order(SPLIT4, 64, 640, 256) == by_items


def test_edges():
    alone = lib().forward_alone
    assert alone(SMALL, 128, 1, 1, 1, 256) and alone(SMALL, 128, 64, 32, 1280, 256)
    assert not alone(SMALL, 128, 65, 1, 64, 256) and not alone(SMALL, 128, 1, 33, 64, 256) and not alone(SMALL, 128, 1, 1, 1281, 256)
    assert not alone(SMALL, 128, 0, 1, 1, 256)                                           # (an empty call lists nothing)
    assert not alone(WIDE, 128, 1, 1, 8, 256)
    assert alone(SMALL, 64, 1, 1, 1920, 256) and alone(SPLIT4, 128, 1, 1, 640, 256) and not alone(SPLIT4, 128, 1, 1, 641, 256)
