"""Lists of middling mean length: the forward's wide form works them whatever the lengths are, told by the number of tiles, and O and LSE are bit for bit those
of the same items in a call with many more rows and keys that no item has, whose mean leaves no other form.  (The form of short documents takes its running
maximum from 32 keys at a time instead of 64: an error of O up to 4 % larger.)  And rows of every head against float32 attention."""
import copy

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LONG = 1600          # rows per item in the larger call


def _in_a_larger_call(ra, torch, fcp):
    big = copy.copy(ra)
    big.tq = big.tkv = max(LONG * ra.n_work, ra.tq, ra.tkv)
    more = lambda t: torch.cat([t, torch.zeros(big.tq - t.shape[0], *t.shape[1:], dtype=t.dtype, device=t.device)])
    big.q, big.d_o, big.k, big.v = (more(t) for t in (ra.q, ra.d_o, ra.k, ra.v))
    nb = fcp.fcp_scratch_bytes(fcp.binding.FCP_SCRATCH_FWD, big.tq, big.tkv, ra.hq, ra.hkv, ra.D, ra.n_work, ra.n_parts)
    big.scratch_f = torch.empty(nb, dtype=torch.uint8, device=ra.device)
    big._alloc_outputs()
    return big


@pytest.mark.parametrize("lens,deg,rank,hq,hkv", [
    ([700 + 37 * i for i in range(24)], 1, 0, 32, 8),
    ([700 + 37 * i for i in range(24)], 1, 0, 40, 8),      # one head per unit
    ([9000] + [650] * 12, 1, 0, 32, 8),                    # one document takes most of the time
    ([8500] + [900] * 46, 1, 0, 8, 1),                     # few heads, a loop longer than a CU's share
    ([4200, 900, 1100, 1000] * 5, 2, 1, 32, 8),            # sharded
])
@pytest.mark.parametrize("how", ["direct", "partial", "running"])
def test_the_wide_form_works_them(lens, deg, rank, hq, hkv, how):
    import torch
    import paper_2602_21788_amd as fcp
    from paper_2602_21788_amd.rank import RankAttention
    D = 128
    ra = RankAttention(lens, [deg if n >= 4200 else 1 for n in lens], rank, hq, hkv, D)
    ra.set_random_inputs(len(lens))
    big = _in_a_larger_call(ra, torch, fcp)
    print(f"middling lists: {len(lens)} sequences over {deg} ranks, {hq}/{hkv} heads, {how}", flush=True)
    for r in (ra, big):
        r.scratch_f.fill_(0xAB)
        for t in (r.o, r.lse, r.o_part, r.lse_part):
            t.fill_(float("nan"))
        {"direct": r.forward_direct, "partial": r.forward, "running": r.forward_running}[how]()
    torch.cuda.synchronize()
    rows = 256 // (2 if (hq // hkv) % 2 == 0 else 1)
    items = ra.work if how != "running" else ra.work[ra.work["step"] == ra.work["step"].max()]      # (running: the list of its last call)
    for r in (ra, big):
        assert fcp.fcp_scratch_status(r.scratch_f) == (sum(-(-int(n) // rows) for n in items["q_len"]), 0)
    assert torch.equal(ra.o, big.o[:ra.tq]) and torch.equal(ra.lse, big.lse[:, :ra.tq])
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
