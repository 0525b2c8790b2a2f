"""The first batch's mean map (nothing accumulated yet) and the accumulation into a given map, at sizes around the
tiles' edges, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2012_02030_amd import binding as ap

pytestmark = pytest.mark.gpu


def start_on_nan(Q, K, causal, weight, lse=None):
    """ap_start_attention_maps on a map full of NaN: every entry has to be written."""
    (B, H, Lq, D), Lk = Q.shape, K.shape[2]
    abar = torch.full((H, Lq, Lk), float("nan"), device="cuda")
    ws_bytes = ap.ap_attention_maps_workspace_bytes(B, H, Lq)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    status = ap.lib().ap_start_attention_maps(
        Q.data_ptr(), K.data_ptr(), lse.data_ptr() if lse is not None else None, ap.AP_BF16, B, H, Lq, Lk, D,
        ap._strides3(Q), ap._strides3(K), int(causal), 0.0, weight, abar.data_ptr(), ws.data_ptr(), ws_bytes,
        int(torch.cuda.current_stream().cuda_stream))
    assert status == ap.AP_OK
    torch.cuda.synchronize()
    return abar


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
    first = ap.ap_accumulate_attention_maps(Q.cuda(), K.cuda(), causal=causal, weight=w)
    Qd, Kd = Q.cuda(), K.cuda()
    assert torch.equal(start_on_nan(Qd, Kd, causal, w), first)
    scores = Q.double() @ K.double().transpose(-1, -2) / D ** 0.5
    if causal:
        scores.masked_fill_(torch.ones(Lq, Lk, dtype=torch.bool).triu(Lk - Lq + 1), float("-inf"))
    lse = scores.logsumexp(-1).float().cuda()
    with_lse = start_on_nan(Qd, Kd, causal, w, lse)
    assert torch.equal(with_lse, ap.ap_accumulate_attention_maps(Qd, Kd, causal=causal, weight=w, lse=lse))
    assert float((with_lse - first).abs().max()) <= 1e-5 * B             # finite, too
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


@pytest.mark.parametrize("order", ["rising", "falling", "last", "far below"])
@pytest.mark.parametrize("Lq,Lk,D,causal", [(130, 515, 64, False), (257, 257, 128, True), (65, 200, 32, False)])
def test_rows_whose_largest_scores_come_late(order, Lq, Lk, D, causal):
    """The row sums are taken relative to an earlier maximum until a tile's sum outgrows it: scores that rise with
    the key, jump at the last one, or start far above or below all others."""
    g = torch.Generator().manual_seed(7)
    Q, K = torch.randn(2, 2, Lq, D, generator=g), torch.randn(2, 2, Lk, D, generator=g)
    Q[..., 0] = 8.0                                                    # key[0] moves every score by sqrt(D) / D * 8
    ramp = torch.linspace(-60, 60, Lk) * D ** 0.5 / 8
    K[..., 0] = {"rising": ramp, "falling": -ramp, "last": torch.where(torch.arange(Lk) == Lk - 1, 90.0, 0.0),
                 "far below": torch.where(torch.arange(Lk) < 64, -90.0, 0.0)}[order]
    Q, K = Q.to(torch.bfloat16), K.to(torch.bfloat16)
    ref = 2 * oracle.mean_attention_map(Q.double().numpy(), K.double().numpy(), causal=causal)
    got = ap.ap_accumulate_attention_maps(Q.cuda(), K.cuda(), causal=causal, weight=1.0).double().cpu().numpy()
    # a score of up to 130 in magnitude, formed in 32 bits from D products, is off by up to a few 2^-24 * 130
    assert np.abs(got - ref).max() <= 2 * 1e-4
    assert np.abs(got.sum(-1) - ref.sum(-1)).max() <= 2 * 1e-4


@pytest.mark.parametrize("level", [-8.0, -200.0])
@pytest.mark.parametrize("first", [64, 70, 128])
@pytest.mark.parametrize("Lq,Lk,D,causal", [(130, 515, 64, False), (100, 260, 128, True), (65, 200, 32, False)])
def test_rows_whose_first_scores_overflow(first, level, Lq, Lk, D, causal):
    """Finite padding rows whose products overflow: every query's first 64 scores and more are -inf, the others ordinary or
    (level -200) so low that their exponentials vanish against any reference but their own maximum."""
    g = torch.Generator().manual_seed(9)
    Q, K = torch.randn(2, 2, Lq, D, generator=g), torch.randn(2, 2, Lk, D, generator=g)
    Q[..., 0] = 8.0                                                    # key[0] moves every score by sqrt(D) / D * 8
    K[..., 0] = torch.where(torch.arange(Lk) < first, -3e38, level * D ** 0.5 / 8)
    Q, K = Q.to(torch.bfloat16), K.to(torch.bfloat16)
    ref = 2 * oracle.mean_attention_map(Q.double().numpy(), K.double().numpy(), causal=causal)
    got = ap.ap_accumulate_attention_maps(Q.cuda(), K.cuda(), causal=causal, weight=1.0).double().cpu().numpy()
    assert np.isfinite(got).all() and (got[..., :first] == 0).all()
    # a score of up to 210 in magnitude, formed in 32 bits from D products, is off by up to a few 2^-24 * 210
    assert np.abs(got - ref).max() <= 2 * 1e-4
    assert np.abs(got.sum(-1) - ref.sum(-1)).max() <= 2 * 1e-4


@pytest.mark.parametrize("Lq,Lk", [(516, 516), (300, 523), (513, 900)])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_first_batch_with_tiles_hidden_as_a_whole(Lq, Lk, D):
    """Their zeros come from other workgroups than the visible tiles (D <= 64) or from the same (D = 128); rows that start
    16-byte aligned, and rows that do not."""
    test_first_batch_and_accumulation(2, 2, Lq, Lk, D, True)


@pytest.mark.parametrize("B,H,Lq,Lk,D,causal", [
    (1, 2, 40, 40, 32, False), (2, 2, 64, 40, 32, False), (3, 1, 33, 100, 32, True), (4, 2, 17, 36, 32, True),
    (5, 2, 130, 260, 32, True), (3, 2, 20, 132, 128, True), (2, 2, 100, 20, 64, False), (2, 1, 260, 131, 64, False),
])
def test_tiles_that_are_mostly_outside_the_map(B, H, Lq, Lk, D, causal):
    """Fewer queries or keys than a tile has, and tiles cut by the map's end or the causal limit, with rows of the map that
    start 16-byte aligned and rows that do not; odd and even numbers of examples."""
    test_first_batch_and_accumulation(B, H, Lq, Lk, D, causal)
