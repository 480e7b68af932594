"""Direct forward of sharded lists whose items are joined (rows with one unit over all ring steps) or stay as they are: against partial results and merge,
with a row or a key too few for a run, spans, and items in any order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,deg,rank,hq,hkv,D,spans,how,merged", [
    ([8000], 2, 1, 32, 8, 128, None, "", False),               # every row has one unit, no row is merged
    ([8000], 2, 1, 32, 8, 128, None, "shuffled", False),
    ([8000], 3, 2, 32, 8, 128, [(0, 2500, 400), (0, 5200, 577)], "", False),
    ([6000, 300, 2500, 41], 3, 0, 40, 8, 128, None, "shuffled", False),
    ([8003], 3, 1, 32, 8, 64, None, "", False),
    ([8000], 2, 1, 32, 8, 128, None, "gap", True),              # a key too few between two segments: no run
    ([8000], 2, 1, 32, 8, 128, None, "twice", True),            # a key in two items
    ([12000], 4, 2, 8, 8, 128, None, "", True),                 # few heads: loops too long
])
def test_joined_items(lens, deg, rank, hq, hkv, D, spans, how, merged):
    import torch
    import paper_2602_21788_amd as fcp
    from paper_2602_21788_amd.rank import RankAttention
    ra = RankAttention(lens, [min(deg, max(1, n // 1000)) for n in lens], rank, hq, hkv, D, spans=spans)
    ra.set_random_inputs(sum(lens))
    print(f"joined items: {lens} over {deg} ranks, rank {rank}, {hq}/{hkv} heads, {D} channels, spans {spans}, {how}", flush=True)
    work = ra.work.copy()
    if how == "shuffled":
        work = work[np.random.default_rng(1).permutation(len(work))]
    else:
        at = [i for i in range(len(work)) if work[i]["k_seq_start"][0] > 0]
        for i in at if how == "gap" else []:
            work["k_seq_start"][i][0] += 1
            work["k_len"][i][0] -= 1
        for i in at if how == "twice" else []:
            work["k_seq_start"][i][0] -= 1
            work["k_len"][i][0] += 1
    ra.work_d = torch.from_numpy(np.ascontiguousarray(work).view(np.uint8).copy()).to(ra.device)
    ra.forward()
    o, lse = ra.o.float(), ra.lse.clone()
    for t in (ra.o, ra.lse, ra.o_part, ra.lse_part):
        t.fill_(float("nan"))
    ra.forward_direct()
    torch.cuda.synchronize()
    tiles, rejected = fcp.fcp_scratch_status(ra.scratch_f)
    assert rejected == 0
    # (bf16 rounds O once; the largest value bounds every row's)
    assert not bool(ra.o.isnan().any()) and float((ra.o.float() - o).abs().max()) <= 2.0 ** -7 * float(o.abs().max())
    assert float((ra.lse - lse).abs().max()) <= 1e-5
    # rows that are merged have partial results
    assert bool((ra.lse_part > float("-inf")).any()) == merged
