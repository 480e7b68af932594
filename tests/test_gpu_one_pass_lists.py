"""GPU parity of the one-pass backward on lists that callers write themselves."""
import numpy as np
import pytest

import listed
from parity import TOL_BF16_REL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("family", ["plain", "direct"])
def test_rows_of_one_sequence_in_many_items(family):
    """32 items of 128 rows of one sequence, each with all keys up to its last row: the items share their keys, and the key tiles of all
    of them (528) are several times those of the sequence."""
    import paper_2602_21788_amd.binding as B
    lens, hq, hkv, D = [4096], 8, 8, 128
    items = [(0, r, 128, [(0, r + 128)]) for r in range(0, 4096, 128)]
    q, k, v, do = listed.draw(lens, hq, hkv, D, 11)
    lse, delta, ref = listed.reference(lens, items, q, k, v, do, D ** -0.5)
    print(f"rows of one sequence in {len(items)} items, {family}", flush=True)
    got, scratch = listed.run_backward(B, family, lens, listed.work_list(B, lens, items), q, k, v, do, lse, delta, D ** -0.5)
    assert B.fcp_scratch_status(scratch) == (528, 0) and listed.backward_path(scratch) == listed.ONE_PASS
    listed.check(got, ref, TOL_BF16_REL, family)


@pytest.mark.parametrize("what", ["k", "v", "q"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_rows_do_not_see_what_later_keys_hold(what, bad):
    """A key row or value row that is not finite reaches only the dQ rows that see it (a key row also those of the same 32-row block, through
    the zeros that it is multiplied with), and a query row whose scores are not finite leaves the dV of later keys alone."""
    import torch
    import paper_2602_21788_amd.binding as B
    lens, hq, hkv, D = [300, 77, 160], 8, 8, 128
    items = [(s, 0, n, [(0, n)]) for s, n in enumerate(lens)]
    cu = listed.offsets(lens)
    q, k, v, do = listed.draw(lens, hq, hkv, D, 12)
    lse, delta, ref = listed.reference(lens, items, q, k, v, do, D ** -0.5)
    at = {0: 150, 1: 70, 2: 127}                          # the bad row of each sequence
    for s, j in at.items():
        {"k": k, "v": v, "q": q}[what][cu[s] + j] = bad
        if what == "q":
            lse[:, cu[s] + j] = float("nan")
    print(f"one-pass backward with {bad} in {what}", flush=True)
    for family in ("plain", "direct"):
        got, scratch = listed.run_backward(B, family, lens, listed.work_list(B, lens, items), q, k, v, do, lse, delta, D ** -0.5)
        assert listed.backward_path(scratch) == listed.ONE_PASS
        dq, _, dv = (x.float().cpu() for x in got)
        for s, n in enumerate(lens):
            j = at[s]
            if what == "q":
                a, b = dv[cu[s] + j + 1:cu[s] + n], ref[2][cu[s] + j + 1:cu[s] + n]
            else:
                last = j if what == "v" else j // 32 * 32
                a, b = dq[cu[s]:cu[s] + last], ref[0][cu[s]:cu[s] + last]
                assert not torch.isfinite(dq[cu[s] + j:cu[s] + n]).all()     # (those that see it do)
            assert torch.isfinite(a).all(), (family, s)
            assert float((a - b).abs().max() / b.abs().max()) <= TOL_BF16_REL, (family, s)


def test_status_reports_waits_that_ran_out():
    """A wait for another unit's turn that ran out is not a rejected work item: the status call has an error of its own for it (the header
    word that the kernels count them in is set here by hand)."""
    import torch
    import paper_2602_21788_amd.binding as B
    lens, hq, hkv, D = [300, 200], 8, 8, 128
    items = [(s, 0, n, [(0, n)]) for s, n in enumerate(lens)]
    q, k, v, do = listed.draw(lens, hq, hkv, D, 13)
    lse, delta, _ = listed.reference(lens, items, q, k, v, do, D ** -0.5)
    _, scratch = listed.run_backward(B, "plain", lens, listed.work_list(B, lens, items), q, k, v, do, lse, delta, D ** -0.5)
    assert B.fcp_scratch_status(scratch) == (5, 0)
    scratch[:64].view(torch.int32)[12] = 3
    with pytest.raises(B.FcpError) as e:
        B.fcp_scratch_status(scratch)
    assert e.value.code == B.FCP_ERR_STALLED and "3 waits" in str(e.value)


def test_one_pass_beside_another_streams_work():
    """Blocks of the kernel that start late or unevenly, because another stream's kernels hold CUs, change nothing: not the sums, whichever
    XCD works a queue of units off, and no wait runs out."""
    import torch
    import paper_2602_21788_amd.binding as B
    from paper_2602_21788_amd.rank import RankAttention
    dev = "cuda:0"
    lens = [3000] + [60] * 20                              # 24 of the 44 units of a queue are one chain
    D, hq, hkv = 128, 8, 8
    items = [(s, 0, n, [(0, n)]) for s, n in enumerate(lens)]
    q, k, v, do = listed.draw(lens, hq, hkv, D, 14)
    lse, delta, ref = listed.reference(lens, items, q, k, v, do, D ** -0.5)
    work = listed.work_list(B, lens, items)
    first, scratch = listed.run_backward(B, "plain", lens, work, q, k, v, do, lse, delta, D ** -0.5)
    assert listed.backward_path(scratch) == listed.ONE_PASS
    listed.check(first, ref, TOL_BF16_REL, "alone")
    other = RankAttention([8192], [1], 0, 16, 8, D)
    other.set_random_inputs(3)
    side, mine = torch.cuda.Stream(), torch.cuda.Stream()
    t = [x.to(dev) for x in (q, k, v, do, lse, delta)] + [torch.from_numpy(listed.offsets(lens)).to(dev)]
    work_d = torch.from_numpy(work.view("u1").copy()).to(dev)
    unused = torch.empty_like(t[5])
    for call in range(12):
        got = [torch.zeros_like(x) for x in first]
        torch.cuda.synchronize()
        print(f"one-pass backward beside another stream, call {call}", flush=True)
        for _ in range(3):
            other.forward_direct(stream=side)
        for _ in range(call % 3):                          # (starts at different places of the other stream's work)
            B.fcp_attn_bwd_delta(t[0], t[3], unused, stream=mine)
        B.fcp_attn_bwd_step(*t, work_d, D ** -0.5, *got, scratch, stream=mine)
        torch.cuda.synchronize()
        assert B.fcp_scratch_status(scratch)[1] == 0
        for a, b in zip(got, first):
            assert torch.equal(a, b), call


_SHORT = [int(x) for x in np.random.default_rng(7).integers(20, 120, 59)]


@pytest.mark.parametrize("lens,hq,path", [
    ([90] + _SHORT, 32, listed.ONE_PASS),
    ([1500] + _SHORT[:30] + [40] * 20, 32, listed.SPLIT_KEYS),                       # two passes, key tiles in pieces
    ([4000] + _SHORT[:30], 24, 0),                                                   # two passes, whole tiles
    ([3000] + _SHORT + [100] * 10, 8, listed.ONE_PASS),                              # one query head per KV head: one pass, whatever the lengths
])
@pytest.mark.parametrize("family", ["plain", "direct"])
def test_the_longest_sequence_decides_between_one_pass_and_two(family, lens, hq, path):
    """The mean length is short in all of these lists; the scheduler sees the longest one."""
    import paper_2602_21788_amd.binding as B
    hkv, D = 8, 128
    assert sum(lens) <= 256 * len(lens) and sum(lens) >= 4096
    items = [(s, 0, n, [(0, n)]) for s, n in enumerate(lens)]
    q, k, v, do = listed.draw(lens, hq, hkv, D, 15)
    lse, delta, ref = listed.reference(lens, items, q, k, v, do, D ** -0.5)
    print(f"one pass or two: {len(lens)} sequences, the longest of {max(lens)}, {hq} heads, {family}", flush=True)
    got, scratch = listed.run_backward(B, family, lens, listed.work_list(B, lens, items), q, k, v, do, lse, delta, D ** -0.5)
    assert B.fcp_scratch_status(scratch)[1] == 0 and listed.backward_path(scratch) == path
    listed.check(got, ref, TOL_BF16_REL, family)


def test_a_captured_backward_decides_anew_at_every_replay():
    """The choice between one pass and two is made on the device: a graph replayed on another list of the same size takes that list's way."""
    import torch
    import paper_2602_21788_amd.binding as B
    hq, hkv, D, dev = 32, 8, 128, "cuda:0"
    lists = {}
    for name, lens in (("short", [100] * 45), ("long", [1500] + [60] * 43 + [420])):
        items = [(s, 0, n, [(0, n)]) for s, n in enumerate(lens)]
        q, k, v, do = listed.draw(lens, hq, hkv, D, 16)
        lse, delta, ref = listed.reference(lens, items, q, k, v, do, D ** -0.5)
        lists[name] = ([x.to(dev) for x in (q, k, v, do, lse, delta, torch.from_numpy(listed.offsets(lens)))] +
                       [torch.from_numpy(listed.work_list(B, lens, items).view("u1").copy()).to(dev)], ref)
    t = [x.clone() for x in lists["short"][0]]
    T = t[0].shape[0]
    scratch = listed.scratch_for(B, T, hq, hkv, D, 45)
    shapes = ((T, hq, D), (T, hkv, D), (T, hkv, D))
    acc = [torch.full(s, float("nan"), device=dev) for s in shapes]
    out = [torch.full(s, float("nan"), device=dev, dtype=torch.bfloat16) for s in shapes]

    def backward():
        B.fcp_attn_bwd_step_direct(*t, D ** -0.5, *acc, *out, scratch)
        B.fcp_grad_finalize_direct(*acc, *out, scratch, 45)

    backward()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        backward()
    for name in ("short", "long", "long", "short", "long"):
        tensors, ref = lists[name]
        for a, b in zip(t, tensors):
            a.copy_(b)
        torch.cuda.synchronize()
        print(f"captured backward, {name} list", flush=True)
        graph.replay()
        torch.cuda.synchronize()
        replayed = [x.clone() for x in out]
        assert listed.backward_path(scratch) == (listed.ONE_PASS if name == "short" else listed.SPLIT_KEYS)
        listed.check(replayed, ref, TOL_BF16_REL, name)
        backward()
        torch.cuda.synchronize()
        for a, b in zip(replayed, out):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16)), name


@pytest.mark.parametrize("hq,hkv,segments", [(8, 8, 1), (16, 8, 2), (16, 16, 1), (24, 8, 1)])
@pytest.mark.parametrize("family", ["plain", "direct"])
def test_one_pass_with_full_attention_spans(family, hq, hkv, segments):
    """Spans that cross the borders of 32-row blocks, key groups and key tiles, a sequence that is one span (its tiles all begin at the
    first block) and spans at a sequence's ends: the order of a chain and the blocks that its tiles begin at follow from the mask."""
    import paper_2602_21788_amd.binding as B
    D = 128
    lens = [300, 1, 129, 513, 260, 64, 400] + [150] * (19 if hq == 24 else 2)        # (three heads per KV head: 256 key tiles at least)
    spans = [(0, 20, 200), (2, 127, 2), (3, 0, 513), (4, 0, 40), (4, 120, 20), (4, 250, 10), (6, 31, 2), (6, 95, 66), (6, 255, 140)]
    items = [(s, 0, n, [(0, n)] if segments == 1 or n < 4 else [(n // 3, n - n // 3), (0, n // 3)]) for s, n in enumerate(lens)]
    q, k, v, do = listed.draw(lens, hq, hkv, D, 17)
    lse, delta, ref = listed.reference(lens, items, q, k, v, do, D ** -0.5, spans)
    print(f"one-pass backward with spans: {hq}/{hkv} heads, {segments} segments, {family}", flush=True)
    got, scratch = listed.run_backward(B, family, lens, listed.work_list(B, lens, items), q, k, v, do, lse, delta, D ** -0.5, spans=spans)
    assert B.fcp_scratch_status(scratch)[1] == 0 and listed.backward_path(scratch) == listed.ONE_PASS
    listed.check(got, ref, TOL_BF16_REL, family)


@pytest.mark.parametrize("family", ["plain", "direct"])
def test_one_pass_with_costs_of_several_blocks_in_one_bucket(family):
    """An item of more than 2048 blocks of rows: the scheduler's list is sorted by cost in steps of two blocks, and the chain's order follows
    it.  A span makes key tiles of one item begin at adjacent blocks, so that tiles of unequal cost share a bucket; two segments whose
    neighbouring tiles do are the other way to that."""
    import torch
    import paper_2602_21788_amd.binding as B
    dev, hq, hkv, D, rows = "cuda:0", 8, 8, 128, 65610                   # 2051 blocks
    short = [int(x) for x in np.random.default_rng(8).integers(20, 60, 329)]
    lens = [rows] + short
    spans = [(0, 32, 1000)]                                              # tile 0 begins at block 0, tiles 1 .. 8 at block 1
    segs = [(0, 2710), (2720, 2300)]                                     # the last tile of the first one begins at block 84, the next at 85
    items = [(0, 0, rows, segs)] + [(s, 0, n, [(0, n)]) for s, n in enumerate(lens) if s > 0]
    q, k, v, do = listed.draw(lens, hq, hkv, D, 19)
    lse, delta = torch.zeros(hq, sum(lens)), torch.zeros(hq, sum(lens))
    ref = [torch.zeros(x.shape) for x in (q, k, v)]
    lse[:, rows:], delta[:, rows:], tail = listed.reference(short, [(s - 1, r, n, g) for s, r, n, g in items[1:]], *(x[rows:] for x in (q, k, v, do)), D ** -0.5)
    for a, b in zip(ref, tail):
        a[rows:] = b
    # the long item in fp32 on the device, its LSE and delta over the listed keys
    keys = torch.cat([torch.arange(a, a + n) for a, n in segs])
    limit = torch.from_numpy(listed.mask_tables([rows], spans)[0]).to(dev)
    hidden = keys.to(dev)[None, :] > limit[:, None]
    for h in range(hq):
        Q, dO, K, V = (x.to(dev).float().contiguous() for x in (q[:rows, h], do[:rows, h], k[keys, h], v[keys, h]))
        S = (Q @ K.T.contiguous() * D ** -0.5).masked_fill_(hidden, float("-inf"))
        L = torch.logsumexp(S, 1)
        P = torch.exp(S - L[:, None])
        del S
        d = ((P @ V) * dO).sum(1)
        lse[h, :rows], delta[h, :rows] = L.cpu(), d.cpu()
        ref[2][keys, h] = (P.T.contiguous() @ dO).cpu()
        dS = P * (dO @ V.T.contiguous() - d[:, None]) * D ** -0.5
        ref[0][:rows, h], ref[1][keys, h] = (dS @ K).cpu(), (dS.T.contiguous() @ Q).cpu()
    print(f"one-pass backward, an item of {rows} rows, {family}", flush=True)
    got, scratch = listed.run_backward(B, family, lens, listed.work_list(B, lens, items), q, k, v, do, lse, delta, D ** -0.5, spans=spans)
    assert B.fcp_scratch_status(scratch)[1] == 0 and listed.backward_path(scratch) == listed.ONE_PASS
    # (gradients of the long item's keys are sums over 65610 rows, those of the short sequences' keys over 60 at most: each part by its own size)
    listed.check([x[:rows] for x in got], [x[:rows] for x in ref], TOL_BF16_REL, f"{family}, long")
    listed.check([x[rows:] for x in got], [x[rows:] for x in ref], TOL_BF16_REL, f"{family}, short")


def test_one_pass_is_no_less_exact_than_two():
    """dQ, dK and dV against 64 bits.  The kernel of two lists sees the same eight heads in two calls of four KV heads, which one pass does not take.
    5 % is left for the rounding of the results, a mean over 340 000 elements and more."""
    import torch
    import paper_2602_21788_amd.binding as B
    lens, hq, hkv, D = [300, 40, 129, 64, 500, 90, 200], 8, 8, 128
    items = [(s, 0, n, [(0, n)]) for s, n in enumerate(lens)]
    q, k, v, do = listed.draw(lens, hq, hkv, D, 20)
    lse, delta, _ = listed.reference(lens, items, q, k, v, do, D ** -0.5)
    ref = [torch.zeros(x.shape, dtype=torch.float64) for x in (q, k, v)]
    cu = listed.offsets(lens)
    for s, n in enumerate(lens):
        r = slice(int(cu[s]), int(cu[s]) + n)
        for h in range(hq):
            Q, K, V, dO = (x[r, h].double() for x in (q, k, v, do))
            P = torch.softmax((Q @ K.T * D ** -0.5).masked_fill(torch.ones(n, n).triu(1) > 0, float("-inf")), 1)
            dP = dO @ V.T
            dS = P * (dP - (P * dP).sum(1, keepdim=True)) * D ** -0.5
            ref[0][r, h], ref[1][r, h], ref[2][r, h] = dS @ K, dS.T @ Q, P.T @ dO
    work = listed.work_list(B, lens, items)
    print("one-pass backward against two passes", flush=True)
    one, scratch = listed.run_backward(B, "direct", lens, work, q, k, v, do, lse, delta, D ** -0.5)
    assert listed.backward_path(scratch) == listed.ONE_PASS
    two = [torch.empty_like(x) for x in one]
    for half in (slice(0, 4), slice(4, 8)):
        got, scratch = listed.run_backward(B, "direct", lens, work, *(x[:, half].contiguous() for x in (q, k, v, do)),
                                           lse[half].contiguous(), delta[half].contiguous(), D ** -0.5)
        assert not listed.backward_path(scratch) & listed.ONE_PASS
        for a, b in zip(two, got):
            a[:, half] = b
    for name, a, b, x in zip(("dQ", "dK", "dV"), one, two, ref):
        e1, e2 = (float((y.double().cpu() - x).norm() / x.norm()) for y in (a, b))
        print(f"  {name} {e1:.3e}, two passes {e2:.3e}", flush=True)
        assert e1 <= 1.05 * e2, name


@pytest.mark.parametrize("family", ["plain", "direct"])
def test_one_pass_inside_larger_buffers_is_not_overrun(family):
    """Every tensor is the front of a larger allocation: the rows after the inputs hold NaN, those after the accumulators and outputs a
    sentinel; the last sequence is no multiple of any tile.  Rows past the end read as zero, stores past it are dropped."""
    import torch
    import paper_2602_21788_amd.binding as B
    dev, hq, hkv, D, pad, sentinel = "cuda:0", 16, 8, 128, 300, 1024.0
    lens = [129, 300, 1, 77, 203]
    items = [(s, 0, n, [(0, n)]) for s, n in enumerate(lens)]
    cpu = listed.draw(lens, hq, hkv, D, 18)
    lse, delta, ref = listed.reference(lens, items, *cpu, D ** -0.5)
    T = cpu[0].shape[0]

    def front(x, fill):
        big = torch.full((T + pad,) + tuple(x.shape[1:]), fill, dtype=x.dtype, device=dev)
        big[:T].copy_(x)
        return big
    ins = [front(x, float("nan")) for x in cpu]
    acc = [front(torch.zeros_like(x), sentinel) for x in ref]
    out = [front(torch.zeros(x.shape, dtype=torch.bfloat16), sentinel) for x in ref]
    guard = [torch.full((hq * T + 4096,), float("nan"), device=dev) for _ in range(2)]     # statistics: [hq, T], NaN behind them
    for g, x in zip(guard, (lse, delta)):
        g[:hq * T].copy_(x.reshape(-1))
    size = B.fcp_scratch_bytes(B.FCP_SCRATCH_BWD, T, T, hq, hkv, D, len(lens), 1)
    room = torch.full((size + 4096,), 165, dtype=torch.uint8, device=dev)
    scratch = room[:size]
    t = [x[:T] for x in ins] + [g[:hq * T].view(hq, T) for g in guard] + [torch.from_numpy(listed.offsets(lens)).to(dev)]
    work_d = torch.from_numpy(listed.work_list(B, lens, items).view("u1").copy()).to(dev)
    print(f"one-pass backward inside larger buffers, {family}", flush=True)
    if family == "plain":
        B.fcp_attn_bwd_step(*t, work_d, D ** -0.5, *[x[:T] for x in acc], scratch)
        got = acc
    else:
        B.fcp_attn_bwd_step_direct(*t, work_d, D ** -0.5, *[x[:T] for x in acc], *[x[:T] for x in out], scratch)
        B.fcp_grad_finalize_direct(*[x[:T] for x in acc], *[x[:T] for x in out], scratch, len(lens))
        got = out
    torch.cuda.synchronize()
    assert B.fcp_scratch_status(scratch)[1] == 0 and listed.backward_path(scratch) == listed.ONE_PASS
    listed.check([x[:T] for x in got], ref, TOL_BF16_REL, family)
    for x in acc + out:
        assert bool((x[T:] == sentinel).all()), "rows after a tensor were written"
    assert bool((room[size:] == 165).all()), "bytes after the scratch were written"
