"""GPU parity of the one-pass backward of many short sequences (blocks of four waves; 2.5 key tiles per CU and more, a mean of 192 rows at most)."""
import numpy as np
import pytest

import listed
from parity import TOL_BF16_REL

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 31, 32, 33, 95, 96, 127, 128, 129, 160, 255, 256, 257, 300]


def _lens(n, lo, hi, seed):
    """More than 10240 rows, 640 key tiles of eight heads."""
    lens = EDGES + [int(x) for x in np.random.default_rng(seed).integers(lo, hi, n)]
    assert sum(lens) >= 10240 and sum(lens) <= 192 * len(lens)
    return lens


def _items(kind, lens):
    items = []
    for s, n in enumerate(lens):
        if kind == "two segments" and n > 8:      # the second one first in memory
            items.append((s, 0, n, [(n // 3, n - n // 3), (0, n // 3)]))
        elif kind == "late keys" and n > 8:       # rows that see no key
            items.append((s, 0, n, [(n // 2, n - n // 2)]))
        elif kind == "shared rows" and n > 8:     # two items with the same rows
            items += [(s, 0, n, [(0, n // 3)])] + ([(s, 0, n, [(n // 3, n - n // 3)])] if s % 2 == 0 else [])
        elif kind == "shared keys" and n > 40:    # two items with the same keys
            items += [(s, 0, n // 2, [(0, n // 2)]), (s, n // 2, n - n // 2, [(0, n)])]
        else:
            items.append((s, 0, n, [(0, n)]))
    return items


@pytest.mark.parametrize("n,lo,hi,hq,hkv,kind,family", [
    (80, 40, 190, 8, 8, "whole", "direct"),       # tiles by their own cost
    (80, 40, 190, 8, 8, "whole", "plain"),
    (270, 8, 140, 24, 8, "whole", "plain"),
    (270, 8, 140, 16, 8, "whole", "direct"),      # 256 tiles and more: an item's tiles one after the other
    (270, 8, 140, 8, 8, "spans", "plain"),
    (270, 8, 140, 16, 16, "two segments", "direct"),
    (80, 40, 190, 8, 8, "late keys", "direct"),
    (270, 8, 140, 8, 8, "shared rows", "direct"),
    (270, 8, 140, 16, 8, "shared rows", "plain"),
    (200, 30, 140, 8, 8, "shared keys", "direct"),
])
def test_many_short(n, lo, hi, hq, hkv, kind, family):
    import torch
    import paper_2602_21788_amd.binding as B
    lens, D = _lens(n, lo, hi, n + hq), 128
    items = _items(kind, lens)
    spans = [(s, m // 4, m // 3) for s, m in enumerate(lens) if m > 20] if kind == "spans" else ()
    q, k, v, do = listed.draw(lens, hq, hkv, D, 31)
    lse, delta, ref = listed.reference(lens, items, q, k, v, do, D ** -0.5, spans)
    work = listed.work_list(B, lens, items)
    print(f"many short sequences: {len(lens)} of {sum(lens)} rows, {hq}/{hkv} heads, {kind}, {family}", flush=True)
    first = None
    for call in range(3):                          # owned rows repeat bit for bit
        got, scratch = listed.run_backward(B, family, lens, work, q, k, v, do, lse, delta, D ** -0.5, spans=spans or None)
        assert B.fcp_scratch_status(scratch)[1] == 0 and listed.backward_path(scratch) == listed.ONE_PASS
        listed.check(got, ref, TOL_BF16_REL, f"{kind}, {family}")
        first = first or got
        if not kind.startswith("shared"):
            assert all(torch.equal(a, b) for a, b in zip(got, first)), call


@pytest.mark.parametrize("longest,path", [(300, listed.ONE_PASS), (6000, 0)])
def test_the_longest_sequence_decides_among_many_short(longest, path):
    import paper_2602_21788_amd.binding as B
    hq, hkv, D = 16, 8, 128
    lens = [int(x) for x in np.random.default_rng(5).integers(20, 120, 220)] + [longest]
    assert sum(lens) >= 10240 and sum(lens) <= 192 * len(lens)
    items = [(s, 0, n, [(0, n)]) for s, n in enumerate(lens)]
    q, k, v, do = listed.draw(lens, hq, hkv, D, 32)
    lse, delta, ref = listed.reference(lens, items, q, k, v, do, D ** -0.5)
    print(f"220 short sequences and one of {longest}", flush=True)
    got, scratch = listed.run_backward(B, "direct", lens, listed.work_list(B, lens, items), q, k, v, do, lse, delta, D ** -0.5)
    assert B.fcp_scratch_status(scratch)[1] == 0 and listed.backward_path(scratch) & listed.ONE_PASS == path
    listed.check(got, ref, TOL_BF16_REL, f"longest {longest}")


@pytest.mark.parametrize("what", ["k", "v"])
def test_rows_do_not_see_what_later_keys_hold(what):
    """A key or value row that holds NaN reaches the dQ rows that see it (a key row also those of the same 32-row block) and no others."""
    import torch
    import paper_2602_21788_amd.binding as B
    hq, hkv, D, dev = 8, 8, 128, "cpu"
    lens = [150] * 80
    items = [(s, 0, n, [(0, n)]) for s, n in enumerate(lens)]
    q, k, v, do = listed.draw(lens, hq, hkv, D, 33)
    lse, delta, ref = listed.reference(lens, items, q, k, v, do, D ** -0.5)
    bad = 70
    {"k": k, "v": v}[what].view(80, 150, hkv, D)[:, bad] = float("nan")
    print(f"many short sequences with NaN in {what}", flush=True)
    got, scratch = listed.run_backward(B, "direct", lens, listed.work_list(B, lens, items), q, k, v, do, lse, delta, D ** -0.5)
    assert listed.backward_path(scratch) == listed.ONE_PASS
    seen = 64 if what == "k" else bad
    a, b = got[0].float().to(dev).view(80, 150, hq, D), ref[0].view(80, 150, hq, D)
    assert not torch.isfinite(a[:, bad:]).all(dim=-1).any()
    assert torch.isfinite(a[:, :seen]).all() and float((a - b)[:, :seen].abs().max() / b[:, :seen].abs().max()) <= TOL_BF16_REL


@pytest.mark.parametrize("lens,path", [
    ([500] * 12, listed.ONE_PASS), ([500] * 11, 0), ([800] * 12, 0),           # a dozen sequences, a mean of 768 rows
    ([900], 0), ([255, 257], listed.ONE_PASS), ([256, 257], 0),                # a mean of 256 rows
])
def test_one_pass_or_two_lists_by_the_mean(lens, path):
    import paper_2602_21788_amd.binding as B
    hq, hkv, D = 8, 8, 128
    items = [(s, 0, n, [(0, n)]) for s, n in enumerate(lens)]
    q, k, v, do = listed.draw(lens, hq, hkv, D, 34)
    lse, delta, ref = listed.reference(lens, items, q, k, v, do, D ** -0.5)
    print(f"one pass or two lists: {lens}", flush=True)
    got, scratch = listed.run_backward(B, "direct", lens, listed.work_list(B, lens, items), q, k, v, do, lse, delta, D ** -0.5)
    assert B.fcp_scratch_status(scratch)[1] == 0 and listed.backward_path(scratch) & listed.ONE_PASS == path
    listed.check(got, ref, TOL_BF16_REL, str(lens))
