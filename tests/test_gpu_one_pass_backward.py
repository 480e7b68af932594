"""GPU parity of the one-pass backward (lists of whole, mostly short sequences, 128 channels per head) at the shapes where its
bookkeeping can go wrong: lengths around the 32-row block and the 128-key tile, items whose first rows see no key, items
without any visible key, and items that share query rows, so that several tiles take turns at the same dQ rows or, where an
item does not own its rows, add with atomics."""
import numpy as np
import pytest

from listed import ONE_PASS, backward_path
from parity import TOL_BF16_REL

pytestmark = pytest.mark.gpu


def _items(kind, lens):
    """[(seq, first row, rows, [(first key, keys), ..]), ..] of whole sequences of the given lengths."""
    items = []
    for s, n in enumerate(lens):
        if kind == "whole" or n < 4:
            items.append((s, 0, n, [(0, n)]))
        elif kind == "late keys":       # rows 0 .. n/2 - 1 see no key
            items.append((s, 0, n, [(n // 2, n - n // 2)]))
        elif kind == "two segments":    # the second one first in memory
            items.append((s, 0, n, [(n // 3, n - n // 3), (0, n // 3)]))
        elif kind == "shared rows":     # two items with the same rows, the first one alone for odd sequences
            items.append((s, 0, n, [(0, n // 3)]))
            if s % 2 == 0:
                items.append((s, 0, n, [(n // 3, n - n // 3)]))
        else:                           # "no keys": an item of early rows with late keys only, then the other rows
            items.append((s, 0, n // 2, [(n // 2, n - n // 2)]))
            items.append((s, n // 2, n - n // 2, [(0, n)]))
    return items


@pytest.mark.parametrize("hq,hkv,kind", [(8, 8, "whole"), (16, 8, "late keys"), (16, 16, "two segments"), (8, 8, "shared rows"),
                                         (24, 8, "no keys"), (16, 8, "whole")])
@pytest.mark.parametrize("family", ["plain", "direct"])
def test_one_pass_backward(family, hq, hkv, kind):
    import torch
    import paper_2602_21788_amd.binding as B
    rng = np.random.default_rng(hq + len(kind))
    lens = [1, 2, 31, 32, 33, 96, 127, 128, 129, 160, 257, 700] + [int(x) for x in rng.integers(3, 200, 25 if hq > 16 else 9)]
    D, scale = 128, 128.0 ** -0.5
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    if kind == "no keys":                # fewer than 256 rows per item, 256 tiles or more
        lens += [150] * (-(-(4096 - T) // 150))
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        T = int(cu[-1])
    items = _items(kind, lens)
    work = np.zeros(len(items), B.WORK_DTYPE)
    for w, (s, row, rows, segs) in zip(work, items):
        w["seq"], w["q_local_off"], w["q_seq_start"], w["q_len"], w["n_seg"] = s, cu[s] + row, row, rows, len(segs)
        for i, (k0, kn) in enumerate(segs):
            w["k_seq_start"][i], w["k_len"][i] = k0, kn
    g = torch.Generator().manual_seed(5)
    q, do = (torch.randn(T, hq, D, generator=g).to(torch.bfloat16) for _ in range(2))
    k, v = (torch.randn(T, hkv, D, generator=g).to(torch.bfloat16) for _ in range(2))
    # fp32 reference on the CPU.  LSE and delta are those of the sequences' full causal attention, so that the weights stay
    # below one; the gradients are the sums over the listed (row, key) pairs.
    lse, delta = torch.zeros(hq, T), torch.zeros(hq, T)
    ref = [torch.zeros(T, hq, D), torch.zeros(T, hkv, D), torch.zeros(T, hkv, D)]
    for s, n in enumerate(lens):
        r = slice(int(cu[s]), int(cu[s]) + n)
        seen = torch.zeros(n, n)
        for ss, row, rows, segs in items:
            if ss == s:
                for k0, kn in segs:
                    seen[row:row + rows, k0:k0 + kn] += 1
        causal = torch.ones(n, n).tril()
        for h in range(hq):
            kv = h // (hq // hkv)
            Q, K, V, dO = q[r, h].float(), k[r, kv].float(), v[r, kv].float(), do[r, h].float()
            S = (Q @ K.T * scale).masked_fill(causal == 0, -np.inf)
            L = torch.logsumexp(S, 1)
            P = torch.exp(S - L[:, None])
            d = ((P @ V) * dO).sum(1)
            lse[h, r], delta[h, r] = L, d
            P = P * (seen * causal)
            dS = P * (dO @ V.T - d[:, None]) * scale
            ref[0][r, h] = dS @ K
            ref[1][r, kv] += dS.T @ Q
            ref[2][r, kv] += P.T @ dO
    dev = "cuda:0"
    t = [x.to(dev) for x in (q, k, v, do)]
    lse, delta, cu_d = lse.to(dev), delta.to(dev), torch.from_numpy(cu).to(dev)
    work_d = torch.from_numpy(work.view(np.uint8).copy()).to(dev)
    scratch = torch.full((B.fcp_scratch_bytes(B.FCP_SCRATCH_BWD, T, T, hq, hkv, D, len(work), 1),), 255, dtype=torch.uint8, device=dev)
    shapes = ((T, hq, D), (T, hkv, D), (T, hkv, D))
    print(f"one-pass backward: {family}, {hq}/{hkv} heads, {kind}, {len(work)} items, {T} rows", flush=True)
    if family == "plain":
        acc = [torch.zeros(s, device=dev) for s in shapes]
        B.fcp_attn_bwd_step(*t, lse, delta, cu_d, work_d, scale, *acc, scratch)
        got = acc
    else:
        acc = [torch.full(s, float("nan"), device=dev) for s in shapes]
        got = [torch.full(s, float("nan"), device=dev, dtype=torch.bfloat16) for s in shapes]
        B.fcp_attn_bwd_step_direct(*t, lse, delta, cu_d, work_d, scale, *acc, *got, scratch)
        B.fcp_grad_finalize_direct(*acc, *got, scratch, len(work))
    torch.cuda.synchronize()
    assert B.fcp_scratch_status(scratch)[1] == 0 and backward_path(scratch) == ONE_PASS
    for name, a, b in zip(("dQ", "dK", "dV"), got, ref):
        a = a.float().cpu()
        assert torch.isfinite(a).all(), name
        err = float((a - b).abs().max() / b.abs().max())
        print(f"  {name} {err:.2e}", flush=True)
        assert err <= TOL_BF16_REL, (name, err)
