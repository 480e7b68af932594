"""The direct forward with one partial slot: no row is merged, and the call itself writes the rows that no (valid) item covers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,hq,hkv,D,drop", [
    ([1, 63, 512, 65], 4, 4, 64, [1]),                # few units
    ([700, 33, 700], 8, 2, 128, [0, 2]),
    ([300], 6, 2, 64, [0]),                           # nothing left
    ([2500, 40, 2500, 129], 32, 8, 128, [1, 3]),      # eight waves in lock step
    ([60] * 200, 8, 1, 128, list(range(0, 200, 3))),  # more items than lanes
])
@pytest.mark.parametrize("how", ["dropped", "rejected"])
def test_rows_without_an_item(lens, hq, hkv, D, drop, how):
    import torch
    import paper_2602_21788_amd as fcp
    from paper_2602_21788_amd.rank import RankAttention
    ra = RankAttention(lens, [1] * len(lens), 0, hq, hkv, D)
    assert ra.n_parts == 1
    ra.set_random_inputs(len(lens))
    ra.forward()                                      # partial results and merge, all items
    o, lse = ra.o.clone(), ra.lse.clone()
    gone = np.zeros(ra.tq, bool)
    work = ra.work.copy()
    for i in drop:
        gone[work[i]["q_local_off"]:work[i]["q_local_off"] + work[i]["q_len"]] = True
        work[i]["seq"] = -5
    if how == "dropped":
        work = np.delete(work, drop)
    gone = torch.from_numpy(gone).to(ra.device)
    o[gone] = 0
    lse[:, gone] = float("-inf")
    for t in (ra.o, ra.lse, ra.o_part, ra.lse_part):
        t.fill_(float("nan"))
    ra.scratch_f.fill_(0xAB)
    ra.work_d, ra.n_work = torch.from_numpy(work.view(np.uint8).copy()).to(ra.device), len(work)
    print(f"one slot: {len(lens)} sequences, {hq}/{hkv} heads, {D} channels, {len(drop)} items {how}", flush=True)
    ra.forward_direct()
    torch.cuda.synchronize()
    assert fcp.fcp_scratch_status(ra.scratch_f)[1] == (len(drop) if how == "rejected" else 0)
    # (the sum over the keys is the same, in the order of the form that the number of items leads to: one bf16 rounding of O)
    assert float((ra.o.float() - o.float()).abs().max()) <= 2.0 ** -7 * max(1.0, float(o.float().abs().max())) and not bool(ra.o[gone].any())
    assert torch.equal(ra.lse == float("-inf"), lse == float("-inf")) and bool(((ra.lse - lse)[:, ~gone].abs() <= 1e-5).all())
