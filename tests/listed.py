"""Helpers of the GPU tests that write their own work lists: items as tuples, the backward of one call on them, and its fp32
reference on the CPU.

An item is (sequence, first row, rows, [(first key, keys), ..]) on whole sequences (the rank holds every row).  Two items may
cover the same rows or the same keys; the gradients are the sums over the listed (row, key) pairs that the mask lets through."""
import numpy as np
import torch


def offsets(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


def work_list(B, lens, items):
    cu = offsets(lens)
    work = np.zeros(len(items), B.WORK_DTYPE)
    for w, (s, row, rows, segs) in zip(work, items):
        w["seq"], w["q_local_off"], w["q_seq_start"], w["q_len"], w["n_seg"] = s, cu[s] + row, row, rows, len(segs)
        for i, (k0, kn) in enumerate(segs):
            w["k_seq_start"][i], w["k_len"][i] = k0, kn
    return work


def mask_tables(lens, spans):
    """(q_limit, k_from) of whole sequences with full-attention spans [(seq, start, len), ..]."""
    cu = offsets(lens)
    limit = np.concatenate([np.arange(n) for n in lens]).astype(np.int32)
    first = limit.copy()
    for s, start, n in spans:
        limit[cu[s] + start:cu[s] + start + n] = start + n - 1
        first[cu[s] + start:cu[s] + start + n] = start
    return limit, first


def draw(lens, hq, hkv, D, seed):
    g = torch.Generator().manual_seed(seed)
    T = int(offsets(lens)[-1])
    q, do = (torch.randn(T, hq, D, generator=g).to(torch.bfloat16) for _ in range(2))
    k, v = (torch.randn(T, hkv, D, generator=g).to(torch.bfloat16) for _ in range(2))
    return q, k, v, do


def reference(lens, items, q, k, v, do, scale, spans=()):
    """lse, delta [hq, T] and (dQ, dK, dV) in fp32.  LSE and delta are those of the sequences' whole attention, so that the weights
    stay below one."""
    cu = offsets(lens)
    (T, hq, D), hkv = q.shape, k.shape[1]
    limit, _ = mask_tables(lens, spans)
    lse, delta = torch.zeros(hq, T), torch.zeros(hq, T)
    grads = [torch.zeros(T, hq, D), torch.zeros(T, hkv, D), torch.zeros(T, hkv, D)]
    for s, n in enumerate(int(x) for x in lens):
        r = slice(int(cu[s]), int(cu[s]) + n)
        allowed = torch.arange(n)[None, :] <= torch.from_numpy(limit[r].astype(np.int64))[:, None]
        listed = torch.zeros(n, n)
        for ss, row, rows, segs in items:
            if ss == s:
                for k0, kn in segs:
                    listed[row:row + rows, k0:k0 + kn] += 1
        listed *= allowed
        for h in range(hq):
            kv = h // (hq // hkv)
            Q, K, V, dO = q[r, h].float(), k[r, kv].float(), v[r, kv].float(), do[r, h].float()
            S = (Q @ K.T * scale).masked_fill(~allowed, -np.inf)
            L = torch.logsumexp(S, 1)
            P = torch.exp(S - L[:, None])
            d = ((P @ V) * dO).sum(1)
            lse[h, r], delta[h, r] = L, d
            P = P * listed
            dS = P * (dO @ V.T - d[:, None]) * scale
            grads[0][r, h] = dS @ K
            grads[1][r, kv] += dS.T @ Q
            grads[2][r, kv] += P.T @ dO
    return lse, delta, grads


def scratch_for(B, T, hq, hkv, D, n_work, device="cuda:0"):
    return torch.full((B.fcp_scratch_bytes(B.FCP_SCRATCH_BWD, T, T, hq, hkv, D, n_work, 1),), 255, dtype=torch.uint8, device=device)


def run_backward(B, family, lens, work, q, k, v, do, lse, delta, scale, spans=None, scratch=None):
    """(dQ, dK, dV) as the GPU has them (fp32 accumulators or, family "direct", bf16 rows) and the scratch buffer."""
    dev = "cuda:0"
    T, hq, D = q.shape
    hkv = k.shape[1]
    t = [x.to(dev) for x in (q, k, v, do)]
    lse, delta, cu = lse.to(dev), delta.to(dev), torch.from_numpy(offsets(lens)).to(dev)
    work_d = torch.from_numpy(work.view(np.uint8).copy()).to(dev)
    tables = [None, None] if spans is None else [torch.from_numpy(x).to(dev) for x in mask_tables(lens, spans)]
    if scratch is None:
        scratch = scratch_for(B, T, hq, hkv, D, len(work))
    shapes = ((T, hq, D), (T, hkv, D), (T, hkv, D))
    if family == "plain":
        got = [torch.zeros(s, device=dev) for s in shapes]
        if spans is None:
            B.fcp_attn_bwd_step(*t, lse, delta, cu, work_d, scale, *got, scratch)
        else:
            B.fcp_attn_bwd_step_mixed(*t, lse, delta, cu, work_d, scale, *tables, *got, scratch)
    else:
        acc = [torch.full(s, float("nan"), device=dev) for s in shapes]
        got = [torch.full(s, float("nan"), device=dev, dtype=torch.bfloat16) for s in shapes]
        B.fcp_attn_bwd_step_direct(*t, lse, delta, cu, work_d, scale, *acc, *got, scratch, q_limit=tables[0], k_from=tables[1])
        B.fcp_grad_finalize_direct(*acc, *got, scratch, len(work))
    torch.cuda.synchronize()
    return got, scratch


ONE_PASS, SPLIT_KEYS, SPLIT_ROWS = 1, 2, 4


def backward_path(scratch):
    """How the last backward on `scratch` was worked: the path word of its key-tile list's header."""
    return int(scratch[:16].cpu().view(torch.int32)[3])


def check(got, ref, tol, label=""):
    for name, a, b in zip(("dQ", "dK", "dV"), got, ref):
        a = a.float().cpu()
        assert torch.isfinite(a).all(), (label, name)
        err = float((a - b).abs().max() / b.abs().max())
        print(f"  {label} {name} {err:.2e}", flush=True)
        assert err <= tol, (label, name, err)
