"""GPU parity of the forward's forms for short documents and small problems (csrc/fcp_attn_fwd_small.hip): rows and keys around the edges of
their tiles (32 rows, 32, 64 and 128 keys), sharded lists, full-attention spans, every way a result leaves the kernel: partial, direct and running.
The form is told by the number of tiles that the scheduler lists: `tile` rows each."""
import numpy as np
import pytest

import fcp_synth as synth
from oracle import attn as oattn
from oracle import plan as oplan

from parity import TOL_BF16_REL, TOL_LSE_ABS, bf16_tensor_to_f64, check_rank, rel_err

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 65, 96, 97, 127, 129, 160, 193, 255]


@pytest.mark.parametrize("lens,deg,rank,hq,hkv,D,tile,spans", [
    # four waves share 32 rows
    ([513, 256, 257, 449], 1, 0, 4, 4, 64, 32, None),
    ([385, 290], 1, 0, 6, 2, 64, 32, [(0, 100, 200), (1, 0, 33)]),
    ([641, 513, 385], 1, 0, 4, 4, 128, 64, None),
    ([641, 513, 385], 1, 0, 8, 2, 128, 32, [(0, 31, 97), (0, 200, 300), (2, 64, 64)]),
    ([2500], 3, 2, 8, 8, 128, 64, None),
    # two waves do
    ([1025, 900, 897, 640, 638], 1, 0, 6, 2, 64, 64, None),
    ([700, 671, 640, 609], 1, 0, 8, 2, 64, 32, None),
    ([1500, 1473], 1, 0, 8, 8, 128, 64, None),
    ([1500, 1473], 1, 0, 8, 2, 128, 32, [(0, 500, 577), (1, 0, 65)]),
    ([4097], 3, 1, 8, 8, 128, 64, None),
    # every wave its own rows
    (EDGES, 1, 0, 6, 2, 64, 128, None),
    (EDGES, 1, 0, 8, 2, 64, 64, [(12, 100, 100)]),
    (EDGES, 1, 0, 8, 8, 128, 128, None),
    (EDGES, 1, 0, 8, 2, 128, 64, [(8, 31, 66), (12, 100, 100)]),
    (EDGES * 9, 1, 0, 32, 8, 128, 64, None),       # enough of them for three blocks per CU
])
def test_forward_forms(lens, deg, rank, hq, hkv, D, tile, spans):
    import torch
    import paper_2602_21788_amd as fcp
    from paper_2602_21788_amd.rank import RankAttention
    deg = [deg] * len(lens)
    wl = synth.custom_workload(lens, deg, hq=hq, hkv=hkv, head_dim=D, seed=sum(lens) + hq)
    q, k, v, _ = synth.draw_qkvdo(wl)
    print(f"forward form of {tile}-row tiles: {len(lens)} sequences, degree {deg[0]}, rank {rank}, {hq}/{hkv} heads, {D} channels, spans {spans}", flush=True)
    # (partial results at head counts where the oracle's per-step partials are quick)
    check_rank(wl, q, k, v, None, rank, backward=False, check_partials=hq <= 8, label=f"tile {tile}", spans=spans)
    ra = RankAttention(wl.seq_lens, wl.cp_degree, rank, hq, hkv, D, wl.softmax_scale, spans=spans)
    ra.set_inputs(q, k, v, None)
    ra.forward_steps_direct()
    assert fcp.fcp_scratch_status(ra.scratch_f)[0] == sum(-(-int(n) // tile) for n in ra.work["q_len"])
    # the running form: the results of one ring step are the initial state of the next
    ra.forward_running()
    torch.cuda.synchronize()
    chunks, _ = oplan.shard_plan(wl.seq_lens, wl.cp_degree, spans=spans)
    rows = oplan.rank_rows(chunks, wl.cu_seqlens, rank)
    sid = None if spans is None else oplan.span_ids(wl.seq_lens, spans)
    O_ref, LSE_ref = oattn.attn_fwd(q, k, v, wl.cu_seqlens, wl.softmax_scale, rows, span_id=sid)
    assert rel_err(bf16_tensor_to_f64(ra.o), O_ref) <= TOL_BF16_REL
    assert np.abs(ra.lse.cpu().numpy().astype(np.float64).T - LSE_ref).max() <= TOL_LSE_ABS
