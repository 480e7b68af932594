"""Forward launches without a list: their blocks find their units from the items themselves.  The same items among rejected ones, too many
for that, go through the scheduler's list: the results are the same up to the order of the sums, in all forms, modes and edges of the rule.  Which of the two
a call went through is told by the path word of its header."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


NO_LIST = 8


def _path(scratch):
    import torch
    return int(scratch[:16].cpu().view(torch.int32)[3])


def _passes(ra, work, torch, fcp):
    """(results, rejected items, path word) of every entry point with that work list, on poisoned buffers."""
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
        out[name] = (ra.o.float(), ra.lse.clone(), ra.lse_part.clone() if name == "partial" else None, fcp.fcp_scratch_status(ra.scratch_f)[1], _path(ra.scratch_f))
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
    ([4600], 4, 1, 32, 8, 128, [(0, 700, 900)], []),        # tiles in the order of their costs, which a mask makes estimates of
    ([260 + 97 * i for i in range(11)], 1, 0, 10, 2, 128, None, [3]),       # the waves share the items
    ([6000, 31, 64, 900, 2000, 129, 1, 700, 333, 65], 1, 0, 6, 2, 64, [(0, 100, 3000), (4, 0, 2000)], []),
    ([90, 8] * 32, 1, 0, 10, 2, 128, None, list(range(0, 64, 5))),
    ([1200, 1200], 1, 0, 8, 1, 64, None, []),               # keys divided among the waves: items in the order of their costs
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
    for name, (o, lse, part, rejected, path) in alone.items():
        o2, lse2, part2, rejected2, path2 = listed[name]
        assert path == NO_LIST and path2 == 0, name
        if name != "running":
            assert rejected == len(drop) and rejected2 == len(drop) + 70, name
        assert torch.equal(lse == float("-inf"), lse2 == float("-inf")), name
        fin = lse2 > float("-inf")
        assert bool(((lse - lse2)[fin].abs() <= 1e-5).all()), name
        # (one bf16 rounding of values below the largest V)
        assert not bool(o.isnan().any()) and float((o - o2).abs().max()) <= 2.0 ** -7 * float(o2.abs().max() + 1e-30), name
        if part is not None:
            assert torch.equal(part == float("-inf"), part2 == float("-inf")) and not bool(part.isnan().any())


@pytest.mark.parametrize("hq,hkv,D,tq,tkv,items,tiles", [
    # (item: rows from, rows, first key, keys, step).  Tiles of 128, 32 and 64 rows; the rows of all items together are more than the keys of the pool
    (4, 4, 64, 512, 512, [(0, 512, 64 * s, 64, s) for s in range(8)], 12),            # the last five items have no tile
    (32, 32, 64, 512, 512, [(0, 512, 64 * s, 64, s) for s in range(8)], 12),          # the same with more units than CUs
    (2, 1, 64, 600, 1200, [(0, 600, 0, 100, 0), (100, 444, 100, 200, 1), (37, 500, 300, 30, 2)], 41),  # the third loses its end
    (8, 4, 128, 700, 60, [(0, 700, 0, 60, 0)], 2),                                       # one slot
])
@pytest.mark.parametrize("how", ["direct", "partial", "running"])
def test_more_tiles_than_the_list_bound(hq, hkv, D, tq, tkv, items, tiles, how):
    """Tiles past the bound, in the order of the list, are not worked: they are counted as rejected and their rows have no result of that item."""
    import torch
    import paper_2602_21788_amd as fcp
    B = fcp.binding
    dev, n_parts = "cuda:0", 1 + max(s for *_, s in items)
    if how == "running" and n_parts > 1:
        items, n_parts = items[:1], 1                       # (one item per row and call)
    g = torch.Generator().manual_seed(tq)
    q = torch.randn(tq, hq, D, generator=g).to(torch.bfloat16)
    k, v = (torch.randn(tkv, hkv, D, generator=g).to(torch.bfloat16) for _ in range(2))
    work = np.zeros(len(items), B.WORK_DTYPE)
    for w, (r, n, k0, kn, s) in zip(work, items):
        w["q_local_off"], w["q_seq_start"], w["q_len"], w["n_seg"], w["step"] = r, r, n, 1, s
        w["k_seq_start"][0], w["k_len"][0] = k0, kn
    from host_rules import forward_plan, lib
    tile, pair, cap, _ = forward_plan(D, hq, hkv, tq, tkv, len(items), n_parts, 1 << 40)
    wanted = [-(-n // tile) for _, n, *_ in items]
    assert lib().forward_alone(1, D, len(items), n_parts, cap * hq // (2 if pair else 1), 256)
    if how != "running":
        assert cap == tiles < sum(wanted)
    # keys that each row sees, through the tiles within the bound
    seen, left = np.zeros((n_parts, tq, tkv), bool), cap
    for (r, n, k0, kn, s), t in zip(items, wanted):
        n = min(n, max(left, 0) * tile)
        left -= t
        seen[s, r:r + n, k0:k0 + kn] = np.arange(k0, k0 + kn)[None] <= np.arange(r, r + n)[:, None]
    G, scale = hq // hkv, 1 / np.sqrt(D)
    sc = torch.stack([q[:, h].double() @ k[:, h // G].double().T.contiguous() for h in range(hq)]).numpy() * scale
    def attend(mask):                                       # O [tq, hq, D], LSE [hq, tq]
        with np.errstate(divide="ignore"):
            p = np.where(mask[None], np.exp(sc), 0.)
            lse = np.log(p.sum(-1))
        w = p / np.maximum(p.sum(-1, keepdims=True), 1e-300)
        return np.stack([w[h] @ v[:, h // G].double().numpy() for h in range(hq)], 1), lse
    o_ref, lse_ref = attend(seen.any(0))
    t = [x.to(dev) for x in (q, k, v)]
    cu, work_d = torch.tensor([0, tkv], dtype=torch.int32, device=dev), torch.from_numpy(work.view(np.uint8).copy()).to(dev)
    scratch = torch.full((B.fcp_scratch_bytes(B.FCP_SCRATCH_FWD, tq, tkv, hq, hkv, D, len(items), n_parts),), 0xAB, dtype=torch.uint8, device=dev)
    o, lse = torch.full((tq, hq, D), float("nan"), device=dev, dtype=torch.bfloat16), torch.full((hq, tq), float("nan"), device=dev)
    o_part, lse_part = torch.full((n_parts, tq, hq, D), float("nan"), device=dev), torch.full((n_parts, hq, tq), float("nan"), device=dev)
    print(f"more tiles than the bound: {hq}/{hkv} heads of {D}, {tq} rows, {tkv} keys, {len(items)} items, {how}", flush=True)
    if how == "direct":
        B.fcp_attn_fwd_step_direct(*t, cu, work_d, n_parts, scale, o_part, lse_part, o, lse, scratch)
        B.fcp_lse_merge_direct(o_part, lse_part, o, lse, tkv, scratch, len(items))
    elif how == "partial":
        B.fcp_attn_fwd_step(*t, cu, work_d, n_parts, scale, o_part, lse_part, scratch)
        for s in range(n_parts):
            assert torch.equal(lse_part[s].cpu() > float("-inf"), torch.from_numpy(attend(seen[s])[1]) > float("-inf")), s
        B.fcp_lse_merge(o_part, lse_part, o, lse)
    else:
        o.zero_(); lse.fill_(float("-inf"))
        B.fcp_attn_fwd_step_running(*t, cu, work_d, scale, o_part[0], lse, scratch, o_out=o)
    torch.cuda.synchronize()
    assert _path(scratch) == NO_LIST
    assert fcp.fcp_scratch_status(scratch) == (min(cap, sum(wanted)), max(sum(wanted) - cap, 0))
    o, lse = o.double().cpu().numpy(), lse.double().cpu().numpy()
    fin = lse_ref > -np.inf
    assert np.array_equal(np.isneginf(lse), ~fin) and np.abs(lse[fin] - lse_ref[fin]).max() <= 1e-3
    # (P and O are rounded to bf16: 2^-9 of the largest value each)
    assert not np.isnan(o).any() and np.abs(o - o_ref).max() <= 2.0 ** -7 * np.abs(o_ref).max()
