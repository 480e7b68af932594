"""Which forward launches do without a list (csrc/fcp_sizes.h): items and slots that a wave holds, and the units it pays for."""
from host_rules import lib

WIDE, SMALL, SPLIT4 = 0, 1, 4


def test_edges():
    alone = lib().forward_alone
    assert alone(SMALL, 128, 1, 1, 1, 256) and alone(SMALL, 128, 64, 32, 1280, 256)
    assert not alone(SMALL, 128, 65, 1, 64, 256) and not alone(SMALL, 128, 1, 33, 64, 256) and not alone(SMALL, 128, 1, 1, 1281, 256)
    assert not alone(SMALL, 128, 0, 1, 1, 256)                                           # (an empty call lists nothing)
    assert not alone(WIDE, 128, 1, 1, 8, 256)
    assert alone(SMALL, 64, 1, 1, 1920, 256) and alone(SPLIT4, 128, 1, 1, 640, 256) and not alone(SPLIT4, 128, 1, 1, 641, 256)
