"""Lists of middling mean length: the scheduler decides from the lengths whether the forward's wide form or that of short documents works them.  The form is told by
the number of tiles; results against the partial form of the same call on the oracle's side (check_rank) where that is quick, else against float32 attention."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,deg,rank,hq,hkv,short", [
    ([700 + 37 * i for i in range(24)], 1, 0, 32, 8, True),
    ([700 + 37 * i for i in range(24)], 1, 0, 40, 8, True),      # one head per unit
    ([9000] + [650] * 12, 1, 0, 32, 8, False),                   # one document takes most of the time
    ([8500] + [900] * 46, 1, 0, 8, 1, False),                    # few heads, a loop longer than a CU's share
    ([4200, 900, 1100, 1000] * 5, 2, 1, 32, 8, None),            # sharded: joined items
])
@pytest.mark.parametrize("how", ["direct", "partial", "running"])
def test_the_lengths_decide(lens, deg, rank, hq, hkv, short, how):
    import torch
    import paper_2602_21788_amd as fcp
    from paper_2602_21788_amd.rank import RankAttention
    D = 128
    ra = RankAttention(lens, [deg if n >= 4200 else 1 for n in lens], rank, hq, hkv, D)
    if ra.n_work == 0:
        pytest.skip("no rows")
    ra.set_random_inputs(len(lens))
    print(f"either form: {len(lens)} sequences over {deg} ranks, {hq}/{hkv} heads, {how}", flush=True)
    ra.scratch_f.fill_(0xAB)
    for t in (ra.o, ra.lse, ra.o_part, ra.lse_part):
        t.fill_(float("nan"))
    {"direct": ra.forward_direct, "partial": ra.forward, "running": ra.forward_running}[how]()
    torch.cuda.synchronize()
    if short is not None and how != "running":
        rows = 256 // (2 if (hq // hkv) % 2 == 0 else 1) // (2 if short else 1)
        assert fcp.fcp_scratch_status(ra.scratch_f) == (sum(-(-int(n) // rows) for n in ra.work["q_len"]), 0)
    # every 97th row of every head in float32
    G = hq // hkv
    worst = 0.
    for c in ra.my_chunks:
        k0 = int(ra.cu[c["seq"]])
        at = torch.arange(0, int(c["len"]), 97, device=ra.device)
        end = int(c["seq_start"]) + int(c["len"])
        k, v = (x[k0:k0 + end].float().repeat_interleave(G, 1).permute(1, 0, 2).contiguous() for x in (ra.k, ra.v))
        q = ra.q[int(c["local_off"]) + at].float().permute(1, 0, 2).contiguous()
        s = torch.bmm(q, k.transpose(1, 2).contiguous()) * ra.scale
        s.masked_fill_(torch.arange(end, device=ra.device)[None, None] > (int(c["seq_start"]) + at)[None, :, None], float("-inf"))
        lse = torch.logsumexp(s, -1)
        o = torch.bmm(torch.exp(s - lse[..., None]), v)
        got = ra.o[int(c["local_off"]) + at].float().permute(1, 0, 2)
        worst = max(worst, float((got - o).abs().max()) / float(o.abs().max()))
        assert float((ra.lse[:, int(c["local_off"]) + at] - lse).abs().max()) <= 1e-3
    assert worst <= 2e-2, worst
