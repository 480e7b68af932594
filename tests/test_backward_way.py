"""Which kernels work a backward, as far as the host decides it from the sizes (bwd_way): each way where it was measured to be the faster one."""
import pytest

from host_rules import EITHER, MANY_SHORT, ONE_PASS, backward_way


@pytest.mark.parametrize("n,mean,hq,hkv,way", [
    # three and a half to four key tiles per CU, one query head per KV head, long sequences: two lists, as below and above
    (1, 13000, 8, 8, 0), (1, 14400, 8, 8, 0), (1, 16384, 8, 8, 0), (1, 17000, 8, 8, 0), (4, 3750, 8, 8, 0), (2, 4096, 16, 16, 0), (8, 1975, 8, 8, 0),
    (12, 768, 8, 8, ONE_PASS), (12, 769, 8, 8, 0), (11, 768, 8, 8, 0),
    # two and a half to four tiles per CU: four-wave blocks for short sequences, the shorter the more heads a step of a chain has
    (110, 95, 40, 8, MANY_SHORT), (80, 133, 40, 8, ONE_PASS), (70, 155, 40, 8, ONE_PASS), (75, 158, 40, 8, ONE_PASS), (80, 133, 64, 8, ONE_PASS),
    (85, 132, 24, 8, MANY_SHORT), (70, 155, 24, 8, ONE_PASS), (75, 158, 32, 8, ONE_PASS), (70, 155, 16, 8, ONE_PASS), (75, 158, 16, 8, MANY_SHORT),
    (64, 164, 8, 8, ONE_PASS), (75, 158, 8, 8, MANY_SHORT), (35, 155, 16, 16, ONE_PASS),
    # from four on, and below two and a half
    (100, 190, 32, 8, MANY_SHORT), (200, 130, 40, 8, MANY_SHORT), (1000, 128, 32, 8, MANY_SHORT), (200, 200, 32, 8, ONE_PASS), (60, 100, 40, 8, ONE_PASS),
])
def test_way(n, mean, hq, hkv, way):
    got = backward_way(hq, hkv, 128, n * mean, n * mean, n)
    assert got & (ONE_PASS | MANY_SHORT) == (way | ONE_PASS if way else 0)
    assert not way & MANY_SHORT or got & EITHER
    for other in (backward_way(hq, hkv, 64, n * mean, n * mean, n), backward_way(hq, hkv, 128, n * mean // 2, n * mean, n),
                  backward_way(hq, hkv, 128, n * mean, n * mean, n, n_cu=32), backward_way(hq // hkv * 6, 6, 128, n * mean, n * mean, n)):
        assert other == 0                                  # 64 channels, sharded lists, a part of the chip, heads that do not divide: two lists
