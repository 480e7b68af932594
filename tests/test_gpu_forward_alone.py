"""Forward launches without a list: their blocks find their units from the items themselves.  The same items among rejected ones, too many
for that, go through the scheduler's list: the results are the same up to the order of the sums, in all forms, modes and edges of the rule."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _passes(ra, work, torch, fcp):
    """(rejected items, results) of every entry point with that work list, on poisoned buffers."""
    ra.work_d, ra.n_work = torch.from_numpy(work.view(np.uint8).copy()).to(ra.device), len(work)
    nb = fcp.fcp_scratch_bytes(fcp.binding.FCP_SCRATCH_FWD, ra.tq, ra.tkv, ra.hq, ra.hkv, ra.D, len(work), ra.n_parts)
    ra.scratch_f = torch.full((nb,), 0xAB, dtype=torch.uint8, device=ra.device)
    out = {}
    for name in ("direct", "partial", "running"):
        for t in (ra.o, ra.lse, ra.o_part, ra.lse_part):
            t.fill_(float("nan"))
        if name == "direct":
            ra.forward_direct()
        elif name == "partial":
            ra.forward()
        else:
            ra.lse.fill_(float("-inf"))
            o_run = torch.zeros(ra.tq, ra.hq, ra.D, device=ra.device)
            ra.o.zero_()
            for s in range(ra.n_parts):
                w = work[(work["step"] == s) | (work["seq"] < 0)]
                d = torch.from_numpy(np.ascontiguousarray(w).view(np.uint8).copy()).to(ra.device)
                fcp.fcp_attn_fwd_step_running(ra.q, ra.k, ra.v, ra.cu_d, d, ra.scale, o_run, ra.lse, ra.scratch_f, o_out=ra.o, q_limit=ra.q_limit_d)
        torch.cuda.synchronize()
        out[name] = (ra.o.float(), ra.lse.clone(), ra.lse_part.clone() if name == "partial" else None, fcp.fcp_scratch_status(ra.scratch_f)[1])
    return out


@pytest.mark.parametrize("lens,deg,rank,hq,hkv,D,spans,drop", [
    ([1], 1, 0, 1, 1, 64, None, []),
    ([512], 1, 0, 4, 4, 64, None, []),
    ([33, 1, 95, 257, 64], 1, 0, 6, 2, 64, [(2, 10, 60), (3, 0, 200)], [1]),
    ([40] * 64, 1, 0, 8, 1, 64, None, [0, 63]),             # as many items as lanes
    ([130, 31] * 15, 1, 0, 8, 8, 128, None, [4]),
    ([2500], 3, 2, 8, 8, 128, None, []),                    # rows with several items, partial slots without keys
    ([1900, 77, 300], 4, 1, 8, 2, 128, [(0, 400, 900), (2, 5, 64)], []),
    ([1500], 5, 4, 16, 8, 64, None, [3]),                   # a slot less for some rows
    ([4097], 3, 1, 32, 8, 128, None, []),                   # several units per resident block
])
def test_without_a_list_and_with_one(lens, deg, rank, hq, hkv, D, spans, drop):
    import torch
    import paper_2602_21788_amd as fcp
    from paper_2602_21788_amd.rank import RankAttention
    ra = RankAttention(lens, [min(deg, n) for n in lens], rank, hq, hkv, D, spans=spans)
    ra.set_random_inputs(sum(lens))
    print(f"forward without a list: {len(lens)} sequences, degree {deg}, rank {rank}, {hq}/{hkv} heads, {D} channels, spans {spans}, {len(drop)} rejected", flush=True)
    work = ra.work.copy()
    assert len(work) <= 64
    work["seq"][drop] = -1
    many = np.zeros(70, ra.work.dtype)                      # (all rejected)
    many["seq"] = -1
    many = np.concatenate([many, work])
    alone, listed = _passes(ra, work, torch, fcp), _passes(ra, many, torch, fcp)
    for name, (o, lse, part, rejected) in alone.items():
        o2, lse2, part2, rejected2 = listed[name]
        if name != "running":
            assert rejected == len(drop) and rejected2 == len(drop) + 70, name
        assert torch.equal(lse == float("-inf"), lse2 == float("-inf")), name
        fin = lse2 > float("-inf")
        assert bool(((lse - lse2)[fin].abs() <= 1e-5).all()), name
        # (one bf16 rounding of values below the largest V)
        assert not bool(o.isnan().any()) and float((o - o2).abs().max()) <= 2.0 ** -7 * float(o2.abs().max() + 1e-30), name
        if part is not None:
            assert torch.equal(part == float("-inf"), part2 == float("-inf")) and not bool(part.isnan().any())
