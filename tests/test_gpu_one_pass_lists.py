"""GPU parity of the one-pass backward on lists that callers write themselves."""
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
    assert B.fcp_scratch_status(scratch) == (528, 0)
    listed.check(got, ref, TOL_BF16_REL, family)
