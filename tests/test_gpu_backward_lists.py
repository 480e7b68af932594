"""GPU parity of the backward that works key tiles and query tiles in one launch (csrc/fcp_attn_bwd_lists.hip): rows and keys around the edges of its
tiles (32-row and 32-key groups, 64-key stages, 64- and 128-row and 128-key units), units worked whole and in halves, heads that divide among
the XCDs and heads that do not."""
import pytest

import fcp_synth as synth

from listed import ONE_PASS, backward_path
from parity import check_rank

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 65, 96, 97, 127, 129, 160, 193, 255, 257]


@pytest.mark.parametrize("lens,deg,rank,hq,hkv,D,spans", [
    (EDGES, 1, 0, 6, 2, 64, None),
    (EDGES, 1, 0, 8, 2, 64, [(8, 31, 66), (12, 100, 100)]),
    (EDGES, 1, 0, 4, 4, 128, None),
    (EDGES, 1, 0, 8, 2, 128, [(8, 31, 66), (12, 100, 100)]),
    ([705, 513, 577], 1, 0, 3, 1, 64, None),                        # halves: 512 keys and more
    ([705, 513, 577], 1, 0, 4, 2, 128, [(0, 31, 97), (2, 64, 64)]),
    ([641, 1153], 1, 0, 32, 4, 64, None),                           # query heads divide among the XCDs, KV heads do not
    ([2050], 3, 1, 16, 8, 64, None),                                # sharded: rows and keys shared by items, two key segments
    ([1931, 70], 2, 1, 8, 4, 128, None),
])
def test_backward_lists(lens, deg, rank, hq, hkv, D, spans):
    deg = [min(deg, n) for n in lens]
    wl = synth.custom_workload(lens, deg, hq=hq, hkv=hkv, head_dim=D, seed=sum(lens) + hq)
    q, k, v, do = synth.draw_qkvdo(wl)
    print(f"backward lists: {len(lens)} sequences, degree {max(deg)}, rank {rank}, {hq}/{hkv} heads, {D} channels, spans {spans}", flush=True)
    res = check_rank(wl, q, k, v, do, rank, backward=True, label="backward lists", spans=spans)
    assert not res["_path"] & ONE_PASS


@pytest.mark.parametrize("lens,hq,hkv,D", [
    ([2048] * 24, 32, 8, 128),          # units of one cost, the last of them in halves
    ([700] * 90, 6, 2, 64),
    ([1500, 900, 1500, 900] * 8, 4, 4, 64),
])
def test_units_in_halves_repeat_bit_for_bit(lens, hq, hkv, D):
    """Which units are worked in halves follows from their place in the list, which does not depend on the run."""
    import torch
    from paper_2602_21788_amd.rank import RankAttention
    ra = RankAttention(lens, [1] * len(lens), 0, hq, hkv, D)
    ra.set_random_inputs(3)
    ra.forward_direct()
    print(f"backward lists, repeated: {len(lens)} sequences, {hq}/{hkv} heads, {D} channels", flush=True)
    for backward in (ra.backward, ra.backward_direct):
        first = None
        for call in range(6):
            if call % 2:
                torch.empty(1 << 28, dtype=torch.uint8, device=ra.device).fill_(call)
            backward()
            torch.cuda.synchronize()
            assert backward_path(ra.scratch_b) == 0
            got = [x.clone() for x in (ra.dq, ra.dk, ra.dv)]
            first = first or got
            for name, a, b in zip(("dQ", "dK", "dV"), got, first):
                assert torch.equal(a.view(torch.int16), b.view(torch.int16)), (backward.__name__, call, name)
