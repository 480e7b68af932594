"""GPU parity where a backward's tiles are split because whole ones would leave the chip idle: few heads or KV heads and
sequences long enough for pieces, with ragged ends, two key segments, a sharded list and full-attention spans.  The pieces add with
atomics, in turn where one item owns the rows, to accumulators that the direct mode clears and converts itself, row by row as the
tiles are split or not."""
import pytest

import fcp_synth as synth

from listed import SPLIT_KEYS, SPLIT_ROWS, backward_path
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


@pytest.mark.parametrize("lens,hq,hkv,D,spans", [
    ([4096], 8, 1, 128, None),
    ([2050, 40, 777], 6, 2, 64, None),
    ([3001, 1500], 4, 2, 128, None),
    ([1700, 300], 5, 1, 64, [(0, 100, 500), (0, 900, 333), (1, 20, 250)]),
])
def test_split_tiles_of_owned_rows_repeat_bit_for_bit(lens, hq, hkv, D, spans):
    """The pieces of a tile take turns where one work item owns the rows: the sums have a fixed order, whatever piece ends first.  (Between the
    calls the blocks' timing differs: other buffers, a cold or a warm cache.)"""
    import torch
    from paper_2602_21788_amd.rank import RankAttention
    wl = synth.custom_workload(lens, [1] * len(lens), hq=hq, hkv=hkv, head_dim=D, seed=sum(lens))
    ra = RankAttention(lens, [1] * len(lens), 0, hq, hkv, D, spans=spans)
    ra.set_inputs(*synth.draw_qkvdo(wl))
    ra.forward_direct()
    print(f"split tiles, repeated: {lens}, {hq}/{hkv} heads, {D} channels, spans {spans}", flush=True)
    for backward in (ra.backward, ra.backward_direct):
        first = None
        for call in range(8):
            if call % 2:
                torch.empty(1 << 28, dtype=torch.uint8, device=ra.device).fill_(call)
            backward()
            torch.cuda.synchronize()
            assert backward_path(ra.scratch_b) & (SPLIT_KEYS | SPLIT_ROWS)
            got = [x.clone() for x in (ra.dq, ra.dk, ra.dv)]
            first = first or got
            for name, a, b in zip(("dQ", "dK", "dV"), got, first):
                assert torch.equal(a.view(torch.int16), b.view(torch.int16)), (backward.__name__, call, name)
