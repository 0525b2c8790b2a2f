"""Calls whose workgroups are too many for one grid dimension (HIP counts its threads in 32 bits): 2^24 workgroups of
256 threads, 2^22 of 1024.  One query and one key, so that the results are known without an oracle: the softmax of
one score is 1, O = V, dV = dO, and dQ = dK = 0 up to the rounding of <dO, V> - <dO, O>."""
import pytest
import torch

from paper_2012_02030_amd import binding as ap

pytestmark = pytest.mark.gpu

B, H, D = 4099, 4096, 32                                     # 16.8 million (example, head) pairs


def _one_key_each(heads):
    return ap.ap_build_layout(torch.ones((heads, 1, 1), dtype=torch.uint8, device="cuda"), 64, 64)


def _randn(dtype, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn((B, H, 1, D), generator=g, device="cuda", dtype=dtype)


def test_fp32_forward_with_more_pairs_than_one_grid_dimension():
    Q, V = _randn(torch.float32, 1), _randn(torch.float32, 2)
    O, lse = ap.ap_sparse_attn_fwd(Q, Q, V, _one_key_each(H))
    assert torch.equal(O, V)
    want = (Q * Q).sum(-1) / D ** 0.5
    assert float((lse - want).abs().max()) <= 1e-5 * float(want.max())


def test_scheduled_backward_with_more_pairs_than_one_grid_dimension():
    lay = _one_key_each(H)
    lt = ap.ap_build_layout_transpose(lay)
    sched, col = ap.ap_build_schedule(lay), ap.ap_build_col_schedule(lay, lt)
    Q, V, dO = _randn(torch.bfloat16, 1), _randn(torch.bfloat16, 2), _randn(torch.bfloat16, 3)
    O, lse = ap.ap_sparse_attn_fwd(Q, Q.clone(), V, lay, sched=sched)
    assert torch.equal(O, V)
    dQ, dK, dV = ap.ap_sparse_attn_bwd(Q, Q.clone(), V, O, dO, lse, lay, lt, sched=sched, col_sched=col)
    assert torch.equal(dV, dO)
    # 32 products of standard normal values in another order, times the largest |Q| (below 7) and the scale
    assert float(dQ.abs().max()) <= 1e-3 and float(dK.abs().max()) <= 1e-3


def test_transpose_and_column_schedule_with_more_workgroups_than_one_grid_dimension():
    heads = (1 << 22) + 5                                    # transpose: a workgroup of 1024 threads per head
    lay = _one_key_each(heads)
    lt = ap.ap_build_layout_transpose(lay)
    at = torch.arange(heads + 1, dtype=torch.int32, device="cuda")
    assert torch.equal(lt.col_ptr, at) and torch.equal(lt.tile_idx, at[:-1]) and not bool(lt.row_idx.any())
    del lay, lt
    heads, Lk = (1 << 18) + 1, 4096                          # column schedule: one of 256 threads per block column
    lay = ap.ap_build_layout(torch.ones((heads, 1, Lk), dtype=torch.uint8, device="cuda"), 64, 64)
    col = ap.ap_build_col_schedule(lay, ap.ap_build_layout_transpose(lay))
    n = heads * (Lk // 64)
    assert bool((col.cnt[:n] == 1).all()) and bool((col.start == -1).all())
    assert not bool(col.cols[:, 0].any()) and bool((col.cols[:, 1:] == 1).all())
    assert bool((col.bitmaps[:, 0] == -1).all()) and not bool(col.bitmaps[:, 1:].any())
