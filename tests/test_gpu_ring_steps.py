"""Direct forward of sharded lists: every ring step of a query chunk has its own partial result, with a running maximum of its own, and O and LSE are bit for bit
those of the call that keeps all partial results and merges them; with a key too few or a key twice, spans, and items in any order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NO_LIST = 8          # path word of a launch without a list


@pytest.mark.parametrize("lens,deg,rank,hq,hkv,D,spans,how,no_list", [
    ([8000], 2, 1, 32, 8, 128, None, "", False),
    ([8000], 2, 1, 32, 8, 128, None, "shuffled", False),
    ([8000], 3, 2, 32, 8, 128, [(0, 2500, 400), (0, 5200, 577)], "", False),
    ([6000, 300, 2500, 41], 3, 0, 40, 8, 128, None, "shuffled", False),
    ([8003], 3, 1, 32, 8, 64, None, "", False),
    ([8000], 2, 1, 32, 8, 128, None, "gap", False),                    # a key too few between two segments
    ([8000], 2, 1, 32, 8, 128, None, "twice", False),                  # a key in two items
    ([12000], 4, 2, 8, 8, 128, None, "", True),                        # few heads: a launch without a list
    ([2500], 3, 2, 8, 8, 128, None, "shuffled", True),                 # the same
])
def test_steps_have_their_own_results(lens, deg, rank, hq, hkv, D, spans, how, no_list):
    import torch
    import paper_2602_21788_amd as fcp
    from paper_2602_21788_amd.rank import RankAttention
    ra = RankAttention(lens, [min(deg, max(1, n // 800)) for n in lens], rank, hq, hkv, D, spans=spans)
    ra.set_random_inputs(sum(lens))
    print(f"ring steps: {lens} over {deg} ranks, rank {rank}, {hq}/{hkv} heads, {D} channels, spans {spans}, {how}", flush=True)
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
    o, lse, part = ra.o.clone(), ra.lse.clone(), ra.lse_part.clone()
    for t in (ra.o, ra.lse, ra.o_part, ra.lse_part):
        t.fill_(float("nan"))
    ra.forward_direct()
    torch.cuda.synchronize()
    assert fcp.fcp_scratch_status(ra.scratch_f)[1] == 0
    assert (int(ra.scratch_f[:16].cpu().view(torch.int32)[3]) == NO_LIST) == no_list
    assert torch.equal(ra.o, o) and torch.equal(ra.lse, lse)
    # rows of several items have the partial results of each
    n = np.zeros(ra.tq, int)
    for w in work:
        n[w["q_local_off"]:w["q_local_off"] + w["q_len"]] += 1
    several = torch.from_numpy(n > 1).to(ra.device)
    assert bool(several.any()) and torch.equal(ra.lse_part[..., several], part[..., several])
