"""The shard plan's order and places where its ranks are numbered densely or searched (base ranks far apart), with chunks that
are empty and with full-attention spans."""
import numpy as np
import pytest

import paper_2602_21788_amd as fcp
from oracle import plan as oplan


@pytest.mark.parametrize("gap", [0, 1, 40, 100003, 400000000])
@pytest.mark.parametrize("spans", [False, True])
def test_plan_with_base_ranks_apart(gap, spans):
    rng = np.random.default_rng(gap % 1000 + spans)
    lens = rng.integers(1, 70, 40).astype(np.int32)
    deg = rng.integers(1, 9, 40).astype(np.int32)        # some sequences have fewer tokens than chunks
    base = (rng.integers(0, 5, 40) * gap + rng.integers(0, 4, 40)).astype(np.int32)
    sp = [(k, int(n) // 3, int(n) // 3) for k, n in enumerate(lens) if n >= 3 and k % 2] if spans else None
    chunks, work = fcp.fcp_shard_plan(lens, deg, base) if sp is None else fcp.fcp_shard_plan_mixed(lens, deg, sp, base)
    ochunks, owork = oplan.shard_plan(lens, deg, base, sp)
    assert chunks.tobytes() == np.ascontiguousarray(ochunks).tobytes()
    assert work.tobytes() == np.ascontiguousarray(owork).tobytes()
