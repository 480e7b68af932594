"""Performance cases of the rank-local attention path: what a training or evaluation program has one CP rank do, through
the package's public entry points, over the range of batch layouts, head layouts, sizes and masks the library takes.

A case is one call pattern ("path") on one batch layout:

  infer   forward only, direct entry points (evaluation, prefill, activation recomputation)
  train   forward and backward of a layer, direct entry points (a rank that holds its whole work list)
  plain   forward and backward through partial results, merge and fp32 accumulators (the C ABI's basic form)
  ring    one call per ring step with the running merge, gradients accumulated per step (a real ring, where each step
          waits for its key/value block)
  plan    host only: pack a micro-batch into groups, choose the CP degrees, emit the shard plan

Tensors are N(0, 1) bf16 from the seed: what queries, keys, values and cotangents look like after normalisation layers.
The batch layout belongs to the case (a fixed `lens_seed`), so that the work of a case does not depend on the seed.
"""
import math

import numpy as np
import torch

import paper_2602_21788_amd as fcp
from paper_2602_21788_amd.rank import RankAttention

IMAGE_TOKENS = 576          # one image: a 24 x 24 grid of patches that see each other in full
COST_MODEL = (2.1e-12, 3.0e-9, 2.0e-5, 1.5e-9, 1.0e-5)   # seconds per token^2, per token, per group, per exchanged token, per ring
# (query heads, KV heads): multi-head, grouped with even and odd group sizes, one KV head
HEADS = [(4, 4), (8, 8), (6, 2), (10, 2), (8, 1), (32, 8), (40, 8)]


def listed():
    return [
        # the smallest call: one short prompt, forward only; launches and latency count
        {"name": "infer_512_d64", "path": "infer", "layout": "one", "tokens": 512, "n_seqs": 1, "degree": 1, "rank": 0,
         "hq": 4, "hkv": 4, "head_dim": 64, "images": False, "lens_seed": 0},
        # a small layer of a short-context model sharded over three ranks
        {"name": "train_4k_degree3", "path": "train", "layout": "one", "tokens": 4096, "n_seqs": 1, "degree": 3, "rank": 1,
         "hq": 8, "hkv": 8, "head_dim": 128, "images": False, "lens_seed": 0},
        # evaluation of a packed batch of ragged documents that stay on one rank
        {"name": "infer_packed_16k", "path": "infer", "layout": "packed", "tokens": 16384, "n_seqs": 16, "degree": 1, "rank": 0,
         "hq": 32, "hkv": 8, "head_dim": 128, "images": False, "lens_seed": 1},
        # the ordinary training step: a long-tailed packed micro-batch, the longest documents sharded
        {"name": "train_packed_32k", "path": "train", "layout": "packed", "tokens": 32768, "n_seqs": 24, "degree": 6, "rank": 0,
         "hq": 32, "hkv": 8, "head_dim": 128, "images": False, "lens_seed": 0},
        # the same for a multimodal model: images inside the documents attend in full
        {"name": "train_packed_32k_images", "path": "train", "layout": "packed", "tokens": 32768, "n_seqs": 24, "degree": 6,
         "rank": 0, "hq": 32, "hkv": 8, "head_dim": 128, "images": True, "lens_seed": 2},
        # long-context training: one document over five ranks (not a power of two)
        {"name": "train_131k_degree5", "path": "train", "layout": "one", "tokens": 131072, "n_seqs": 1, "degree": 5, "rank": 2,
         "hq": 32, "hkv": 8, "head_dim": 128, "images": False, "lens_seed": 0},
        # one long video among short captions: the imbalance that flexible degrees are for
        {"name": "train_video_64k", "path": "train", "layout": "video", "tokens": 65536, "n_seqs": 65, "degree": 6, "rank": 0,
         "hq": 40, "hkv": 8, "head_dim": 128, "images": False, "lens_seed": 0},
        # instruction tuning: a thousand short ragged samples in one batch
        {"name": "train_1000_short", "path": "train", "layout": "short", "tokens": 128000, "n_seqs": 1000, "degree": 1, "rank": 0,
         "hq": 32, "hkv": 8, "head_dim": 128, "images": False, "lens_seed": 3},
        # a small model: narrow heads, an odd number of query heads per KV head, odd lengths
        {"name": "train_packed_20k_d64", "path": "train", "layout": "packed", "tokens": 20011, "n_seqs": 30, "degree": 3, "rank": 0,
         "hq": 6, "hkv": 2, "head_dim": 64, "images": False, "lens_seed": 4},
        # a real ring over four ranks: one call per step
        {"name": "ring_32k_degree4", "path": "ring", "layout": "one", "tokens": 32768, "n_seqs": 1, "degree": 4, "rank": 0,
         "hq": 32, "hkv": 8, "head_dim": 128, "images": False, "lens_seed": 0},
        # the basic entry points (partials, merge, accumulators) at an odd degree and length
        {"name": "plain_30k_degree7", "path": "plain", "layout": "one", "tokens": 30011, "n_seqs": 1, "degree": 7, "rank": 3,
         "hq": 32, "hkv": 8, "head_dim": 128, "images": False, "lens_seed": 0},
        # the planner of a global batch on the host
        {"name": "plan_512_on_64", "path": "plan", "layout": "packed", "tokens": 512 * 2500, "n_seqs": 512, "degree": 64, "rank": 0,
         "hq": 32, "hkv": 8, "head_dim": 128, "images": False, "lens_seed": 0},
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One case of the ranges the listed ones stand for, no dearer than the dearest of them."""
    most = max(work(c)["flops"] for c in listed())
    while True:
        path = rng.choice(["infer", "train", "train", "train", "plain", "ring", "plan"])
        hq, hkv = rng.choice(HEADS)
        case = {"path": path, "layout": "one", "tokens": 0, "n_seqs": 1, "degree": 1, "rank": 0, "hq": hq, "hkv": hkv,
                "head_dim": rng.choice([64, 128, 128]), "images": False, "lens_seed": rng.randrange(1 << 20)}
        if path == "plan":
            case["layout"], case["n_seqs"] = "packed", _log_between(rng, 32, 1024)
            case["tokens"] = case["n_seqs"] * _log_between(rng, 300, 6000)
            case["degree"] = rng.choice([8, 16, 24, 32, 64])          # ranks
            return case
        case["layout"] = rng.choice(["one", "packed", "packed", "short", "video"]) if path != "ring" else rng.choice(["one", "packed"])
        if case["layout"] == "one":
            case["tokens"] = _log_between(rng, 300, 131072)
            case["degree"] = rng.randint(1, 8)
            case["rank"] = rng.randrange(case["degree"])
        elif case["layout"] == "packed":
            case["tokens"] = _log_between(rng, 2000, 65536)
            case["n_seqs"] = min(_log_between(rng, 2, 64), case["tokens"] // 64)
            case["degree"] = rng.randint(1, 8)                        # cap; a sequence takes one rank per 4096 tokens
        elif case["layout"] == "video":
            case["tokens"] = _log_between(rng, 16384, 65536)
            case["n_seqs"] = 1 + rng.randint(8, 64)
            case["degree"] = rng.randint(2, 8)
        else:
            case["n_seqs"] = _log_between(rng, 30, 1000)
            case["tokens"] = case["n_seqs"] * rng.randint(40, 160)
        case["images"] = case["layout"] in ("one", "packed") and rng.random() < 0.25
        if work(case)["flops"] <= most:
            return case


# ---- layouts ------------------------------------------------------------------------------------------------------------
def _lens(case):
    """(lengths, degrees) of the case's sequences."""
    rng = np.random.default_rng(case["lens_seed"])
    n, total = case["n_seqs"], case["tokens"]
    if case["layout"] == "one":
        return np.array([total], np.int32), np.array([case["degree"]], np.int32)
    if case["layout"] == "video":               # one long sequence, the rest short captions
        short = rng.integers(128, 513, size=n - 1)
        lens = np.concatenate([[max(total - int(short.sum()), 2048)], short])
        return lens.astype(np.int32), np.array([case["degree"]] + [1] * (n - 1), np.int32)
    if case["layout"] == "short":               # around the mean, between a few tokens and twice the mean
        mean = total // n
        return rng.integers(8, 2 * mean - 7, size=n).astype(np.int32), np.ones(n, np.int32)
    x = rng.lognormal(6.5, 1.2, size=n)         # long-tailed documents, scaled to the token count
    lens = np.maximum((x * (total / x.sum())).astype(np.int64), 16)
    lens[int(np.argmax(lens))] += total - int(lens.sum())
    degree = np.clip((lens + 4095) // 4096, 1, case["degree"])
    return lens.astype(np.int32), degree.astype(np.int32)


def _spans(case, lens):
    """Image spans: every sequence longer than an image spends about a third of its tokens on images."""
    if not case["images"]:
        return None
    rng = np.random.default_rng(case["lens_seed"] + 77)
    spans = []
    for k, n in enumerate(int(x) for x in lens):
        images = int(n * 0.35) // IMAGE_TOKENS
        cuts = np.sort(rng.integers(0, n - images * IMAGE_TOKENS + 1, size=images))   # text tokens before each image
        spans += [(k, int(c) + i * IMAGE_TOKENS, IMAGE_TOKENS) for i, c in enumerate(cuts)]
    return spans


# ---- the interface ----------------------------------------------------------------------------------------------------
def prepare(case, seed):
    if case["path"] == "plan":
        rng = np.random.default_rng(case["lens_seed"])
        n = case["n_seqs"]
        lens = np.clip(rng.lognormal(6.5, 1.2, size=n) * (case["tokens"] / n / 1366.0), 16, case["tokens"] // 4).astype(np.int32)
        # the seed shuffles the documents; the mask factor goes with the document, so that every order makes a plan of one size
        lens = np.random.default_rng(seed).permutation(lens)
        eta = (lens % 97 / 323.0).astype(np.float32)
        ranks = case["degree"]
        # two and a half times the average load per rank: best-fit packing then never needs more ranks than there are
        return {"case": case, "lens": lens, "eta": eta, "ranks": ranks, "per_rank": int(2.5 * int(lens.sum()) / ranks) + 1}
    lens, degree = _lens(case)
    ra = RankAttention(lens, degree, case["rank"], case["hq"], case["hkv"], case["head_dim"], spans=_spans(case, lens))
    ra.set_random_inputs(seed)
    state = {"case": case, "rank": ra}
    if case["path"] == "ring":      # the work items of each ring step, uploaded once per micro-batch
        ra.o_run = torch.empty(ra.tq, ra.hq, ra.D, dtype=torch.float32, device=ra.device)
        state["steps"] = []
        for s in range(ra.n_parts):
            w = np.ascontiguousarray(ra.work[ra.work["step"] == s])
            if len(w):
                state["steps"].append(torch.from_numpy(w.view(np.uint8).copy()).to(ra.device))
    return state


def run(state):
    path = state["case"]["path"]
    if path == "plan":
        plan = fcp.fcp_plan_groups(state["lens"], state["ranks"], state["per_rank"], COST_MODEL, eta=state["eta"])
        degree, base = fcp.fcp_group_shard_args(plan["group_of_seq"], plan["degree"], plan["base_rank"])
        chunks, items = fcp.fcp_shard_plan(state["lens"], degree, base)
        return {"plan": plan, "degree": degree, "base": base, "chunks": chunks.view(np.int32), "items": items.view(np.int32)}
    ra = state["rank"]
    if path == "infer":
        ra.forward_direct()
        return {"o": ra.o, "lse": ra.lse}
    if path == "train":
        ra.forward_direct()
        ra.backward_direct()
    elif path == "plain":
        ra.forward()
        ra.backward()
    else:
        ra.lse.fill_(float("-inf"))
        for w in state["steps"]:
            fcp.fcp_attn_fwd_step_running(ra.q, ra.k, ra.v, ra.cu_d, w, ra.scale, ra.o_run, ra.lse, ra.scratch_f, o_out=ra.o,
                                          q_limit=ra.q_limit_d)
        ra.zero_grads()
        ra.backward_delta()
        for w in state["steps"]:
            if ra.spans is not None:
                fcp.fcp_attn_bwd_step_mixed(ra.q, ra.k, ra.v, ra.d_o, ra.lse, ra.delta, ra.cu_d, w, ra.scale, ra.q_limit_d,
                                            ra.k_from_d, ra.dq_acc, ra.dk_acc, ra.dv_acc, ra.scratch_b)
            else:
                fcp.fcp_attn_bwd_step(ra.q, ra.k, ra.v, ra.d_o, ra.lse, ra.delta, ra.cu_d, w, ra.scale, ra.dq_acc, ra.dk_acc,
                                      ra.dv_acc, ra.scratch_b)
        ra.finalize()
    return {"o": ra.o, "lse": ra.lse, "dq": ra.dq, "dk": ra.dk, "dv": ra.dv}


def work(case):
    if case["path"] == "plan":      # lengths and mask factors in; groups, degrees and some ten records per sequence out
        return {"bytes": float(case["n_seqs"] * (8 + 20 + 10 * 68)), "flops": 0.0}
    lens, degree = _lens(case)
    spans = _spans(case, lens)
    if spans is None:
        chunks, _ = fcp.fcp_shard_plan(lens, degree)
    else:
        chunks, _ = fcp.fcp_shard_plan_mixed(lens, degree, spans)
    mine = chunks[chunks["rank"] == case["rank"]]
    start, n = mine["seq_start"].astype(np.int64), mine["len"].astype(np.int64)
    if spans is None:
        pairs = int((n * start + n * (n + 1) // 2).sum())
    else:
        q_limit, _, _ = fcp.fcp_mask_tables(lens, spans, chunks, case["rank"])
        pairs = int(q_limit.astype(np.int64).sum()) + len(q_limit)
    rows, pool, dim = int(n.sum()), int(lens.sum()), case["head_dim"]
    q_bytes, kv_bytes, stat_bytes = rows * case["hq"] * dim * 2, pool * case["hkv"] * dim * 2, rows * case["hq"] * 4
    flops = pairs * dim * case["hq"]
    if case["path"] == "infer":     # Q, K, V in; O, LSE out
        return {"bytes": float(2 * q_bytes + 2 * kv_bytes + stat_bytes), "flops": 4.0 * flops}
    # and dO in; dQ, dK, dV out
    return {"bytes": float(4 * q_bytes + 4 * kv_bytes + stat_bytes), "flops": 14.0 * flops}


def tolerance(case):
    # plan: whole numbers, and a makespan in double precision; attention: probabilities and results rounded to bf16
    return {"rel": 1e-12, "differ": 0.0} if case["path"] == "plan" else {"rel": 1e-2}
