"""GPU parity where a backward's tiles are split because whole ones would leave the chip idle: few heads or KV heads and
sequences long enough for pieces, with ragged ends, two key segments, a sharded list and full-attention spans.  The pieces add with
atomics to accumulators that the direct mode clears and converts itself, row by row as the tiles are split or not."""
import pytest

import fcp_synth as synth

from listed import SPLIT_KEYS, SPLIT_ROWS
from parity import check_rank

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,deg,rank,hq,hkv,D,spans,path", [
    ([1601], [1], 0, 8, 1, 128, None, SPLIT_KEYS | SPLIT_ROWS),                  # rows and keys in pieces, the last one of a single row
    ([2050, 40, 777], [1, 1, 1], 0, 6, 2, 64, None, SPLIT_KEYS | SPLIT_ROWS),    # an item whose tiles are split among others whose are not
    ([4100], [2], 1, 4, 4, 64, None, SPLIT_ROWS),                   # two items with two key segments each
    ([1700, 300], [1, 1], 0, 5, 1, 64, [(0, 100, 500), (0, 900, 333), (1, 20, 250)], SPLIT_KEYS | SPLIT_ROWS),
])
def test_split_tiles(lens, deg, rank, hq, hkv, D, spans, path):
    wl = synth.custom_workload(lens, deg, hq=hq, hkv=hkv, head_dim=D, seed=sum(lens))
    q, k, v, do = synth.draw_qkvdo(wl)
    print(f"split tiles: {lens} at degree {deg}, rank {rank}, {hq}/{hkv} heads, {D} channels, spans {spans}", flush=True)
    res = check_rank(wl, q, k, v, do, rank, backward=True, check_partials=False, label="split tiles", spans=spans)
    assert res["_path"] == path
