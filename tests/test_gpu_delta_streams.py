"""Delta = rowsum(O dO) where dO is read through the caches and past them: both sides of the line, ragged rows, both widths."""
import pytest

from host_rules import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tq,hq,D,streams", [(1024, 128, 128, False), (1025, 128, 128, True), (2039, 128, 64, False), (8193, 32, 64, True), (33, 3, 64, False)])
def test_delta(tq, hq, D, streams):
    import torch
    import paper_2602_21788_amd as fcp
    assert bool(lib().delta_streams_do(tq, hq, D)) == streams
    g = torch.Generator(device="cuda:0").manual_seed(tq)
    o, do = (torch.randn(tq, hq, D, generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(2))
    delta = torch.full((hq, tq), float("nan"), device="cuda:0")
    print(f"delta: {tq} rows, {hq} heads of {D}", flush=True)
    fcp.fcp_attn_bwd_delta(o, do, delta)
    torch.cuda.synchronize()
    p = o.double() * do.double()
    # (products of bf16 are exact in fp32; a sum of D of them in any order is off by D 2^-24 of the sum of their sizes at most)
    bound = D * 2.0 ** -24 * p.abs().sum(-1).T
    assert bool(((delta.double() - p.sum(-1).T).abs() <= bound).all())
