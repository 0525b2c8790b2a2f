"""The first batch's mean map (nothing accumulated yet) and the accumulation into a given map, at sizes around the
tiles' edges, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2012_02030_amd import binding as ap

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,Lq,Lk,D,causal", [
    (1, 1, 1, 1, 32, True), (2, 3, 31, 33, 64, False), (3, 1, 127, 129, 64, True), (1, 2, 128, 128, 128, True),
    (2, 1, 129, 385, 128, True), (1, 5, 300, 191, 64, False), (2, 2, 4, 700, 32, True), (1, 3, 1030, 1030, 64, True),
])
def test_first_batch_and_accumulation(B, H, Lq, Lk, D, causal):
    g = torch.Generator().manual_seed(Lq * 1000 + Lk)
    Q = torch.randn(B, H, Lq, D, generator=g).to(torch.bfloat16)
    K = torch.randn(B, H, Lk, D, generator=g).to(torch.bfloat16)
    ref = B * oracle.mean_attention_map(Q.double().numpy(), K.double().numpy(), causal=causal)
    w = 0.5
    junk = torch.full((H, Lq, Lk), float("nan"), device="cuda")          # what a fresh map may hold
    del junk
    first = ap.ap_accumulate_attention_maps(Q.cuda(), K.cuda(), causal=causal, weight=w)
    zeroed = ap.ap_accumulate_attention_maps(Q.cuda(), K.cuda(), torch.zeros(H, Lq, Lk, device="cuda"), causal=causal,
                                             weight=w)
    base = torch.randn(H, Lq, Lk, generator=g).cuda()
    onto = ap.ap_accumulate_attention_maps(Q.cuda(), K.cuda(), base.clone(), causal=causal, weight=w)
    torch.cuda.synchronize()
    assert torch.equal(first, zeroed)
    got = first.double().cpu().numpy()
    hidden = np.triu(np.ones((Lq, Lk), bool), Lk - Lq + 1) if causal else np.zeros((Lq, Lk), bool)
    assert (got[:, hidden] == 0).all()
    assert np.abs(got - w * ref).max() <= 1e-5 * B
    # one fused multiply-add per entry onto what was there; hidden entries stay as they are
    assert (onto.cpu().numpy()[:, hidden] == base.cpu().numpy()[:, hidden]).all()
    assert float((onto - (base + first)).abs().max()) <= 1e-6 * float(base.abs().max() + 1)
