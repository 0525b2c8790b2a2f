"""GPU parity of the backward pass (gradients of the masked-attention equation of Section 3.2)
against the fp64 oracle, and of the transposed layout against its definition.

Tolerance: gradients are sums of up to Lk (dQ) or Lq (dK, dV) products whose factors P and dS are
rounded to bf16 (relative 2^-9) before the matrix-core product, the result is rounded to bf16
once more, and delta uses the bf16 O of the forward pass.  With O(1) inputs that gives errors of
a few 1e-3 of the largest gradient entry; the bar (gpu_util.assert_grad_close) is the forward
pass's 2e-2 scaled to the gradient's magnitude, applied per row (every query of dQ, every key of
dK and dV: error <= 2e-2 * max(1, max|oracle row|)) and per tensor, plus a relative Frobenius
error of at most 1e-2 per tensor.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2012_02030_amd import binding as ap
from paper_2012_02030_amd import synth

from gpu_util import assert_grad_close, to_device

pytestmark = pytest.mark.gpu


def transpose_reference(row_ptr, col_idx, H, nQB, nKB):
    cols = [[] for _ in range(H * nKB)]
    for r in range(H * nQB):
        h, qb = divmod(r, nQB)
        for t in range(row_ptr[r], row_ptr[r + 1]):
            cols[h * nKB + col_idx[t]].append((qb, t))
    col_ptr = np.zeros(H * nKB + 1, dtype=np.int32)
    row_idx, tile_idx = [], []
    for c, lst in enumerate(cols):
        col_ptr[c + 1] = col_ptr[c] + len(lst)
        row_idx += [q for q, _ in lst]
        tile_idx += [t for _, t in lst]
    return col_ptr, np.array(row_idx, dtype=np.int32), np.array(tile_idx, dtype=np.int32)


@pytest.mark.parametrize("shape", [(2, 64, 64, 0.5), (3, 200, 330, 0.02), (1, 1000, 70, 0.3), (2, 130, 130, 0.0)])
def test_layout_transpose_matches_definition(shape):
    H, Lq, Lk, density = shape
    mask = synth.random_mask(H, Lq, Lk, density, seed=Lq)
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64)
    lt = ap.ap_build_layout_transpose(lay)
    torch.cuda.synchronize()
    rp, ci, _ = oracle.build_layout(mask, 64, 64)
    nQB, nKB = -(-Lq // 64), -(-Lk // 64)
    col_ptr, row_idx, tile_idx = transpose_reference(rp, ci, H, nQB, nKB)
    nnz = len(ci)
    assert np.array_equal(lt.col_ptr.cpu().numpy(), col_ptr)
    assert np.array_equal(lt.row_idx[:nnz].cpu().numpy(), row_idx)
    assert np.array_equal(lt.tile_idx[:nnz].cpu().numpy(), tile_idx)


@pytest.mark.parametrize("shape", [
    (2, 1, 1, 0.9, 64),                # one tile
    (2, 257, 4097, 0.002, 64),         # 65 block columns: a second workgroup per head with one column
    (2, 100, 2047, 0.05, 16),          # 128 block columns, exactly two workgroups
    (1, 16 * 4096, 40, 0.02, 16),      # as many block rows as the table holds
    (2, 16 * 4097 + 1, 40, 0.02, 16),  # and two more: a second round with its own bits
])
def test_layout_transpose_at_the_edges_of_its_table(shape):
    H, Lq, Lk, density, block = shape
    print("transpose", shape, flush=True)
    mask = synth.random_mask(H, Lq, Lk, density, seed=Lq)
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), block, block)
    lt = ap.ap_build_layout_transpose(lay)
    torch.cuda.synchronize()
    rp, ci, _ = oracle.build_layout(mask, block, block)
    col_ptr, row_idx, tile_idx = transpose_reference(rp, ci, H, -(-Lq // block), -(-Lk // block))
    assert np.array_equal(lt.col_ptr.cpu().numpy(), col_ptr)
    assert np.array_equal(lt.row_idx[:len(ci)].cpu().numpy(), row_idx)
    assert np.array_equal(lt.tile_idx[:len(ci)].cpu().numpy(), tile_idx)


def run_bwd(Q, K, V, dO, mask_np, causal, scale=0.0, per_row=True):
    dq, rq = to_device(Q, "bf16")
    dk, rk = to_device(K, "bf16")
    dv, rv = to_device(V, "bf16")
    dg, rg = to_device(dO, "bf16")
    lay = ap.ap_build_layout(torch.from_numpy(mask_np).cuda(), 64, 64)
    lt = ap.ap_build_layout_transpose(lay)
    O, lse = ap.ap_sparse_attn_fwd(dq, dk, dv, lay, causal=causal, softmax_scale=scale)
    gQ, gK, gV = ap.ap_sparse_attn_bwd(dq, dk, dv, O, dg, lse, lay, lt, causal=causal, softmax_scale=scale)
    torch.cuda.synchronize()
    ref = oracle.masked_attention_backward(rq, rk, rv, mask_np, rg, causal=causal, scale=scale)
    errs = []
    for name, got, want in zip(("dQ", "dK", "dV"), (gQ, gK, gV), ref):
        errs.append(assert_grad_close(name, got.double().cpu().numpy(), want, per_row=per_row)[0])
    return errs


def rand_inputs(seed, B, H, Lq, Lk, D):
    rng = np.random.default_rng([synth.SEED, 4242, seed])
    return tuple(rng.standard_normal(s, dtype=np.float32) for s in
                 ((B, H, Lq, D), (B, H, Lk, D), (B, H, Lk, D), (B, H, Lq, D)))


BWD_CASES = [
    # B, H, Lq, Lk, D, causal, density
    (2, 3, 128, 128, 64, False, 0.5),
    (1, 2, 200, 200, 64, True, 0.3),
    (2, 2, 100, 157, 32, False, 0.3),
    (1, 2, 100, 300, 128, True, 0.2),
    (1, 1, 192, 192, 128, False, 1.0),       # nothing pruned: ordinary attention
    (1, 2, 64, 64, 64, True, 0.05),          # very sparse: empty rows and columns
    (1, 1, 1, 1, 32, False, 1.0),
]


@pytest.mark.parametrize("case", BWD_CASES, ids=lambda c: "B%d_H%d_%dx%d_D%d_%s_%g" % (c[:5] + ("causal" if c[5] else "full", c[6])))
def test_backward_matches_oracle(case):
    B, H, Lq, Lk, D, causal, density = case
    Q, K, V, dO = rand_inputs(Lq + Lk + D, B, H, Lq, Lk, D)
    mask = synth.random_mask(H, Lq, Lk, density, seed=D + Lq)
    run_bwd(Q, K, V, dO, mask, causal)


def test_backward_on_the_structured_masks():
    """C3's band-plus-spikes causal mask (two heads of it) and C2's noisy non-causal one."""
    for name, heads, batch in (("C3", 2, 1), ("C2", 3, 2)):
        cfg = synth.CONFIGS[name]
        mask = np.stack([synth.head_mask(cfg, h) for h in range(heads)]).astype(np.uint8)
        Q, K, V, dO = rand_inputs(7, batch, heads, cfg.Lq, cfg.Lk, cfg.D)
        run_bwd(Q, K, V, dO, mask, cfg.causal)


def test_backward_explicit_scale_and_large_scores():
    """Scores with a standard deviation of 6.4: P is nearly one-hot, so dS = P (dP - delta) is a
    difference of two numbers of size |dO_i| |V_j| ~ 8 that nearly cancel.  delta comes from the
    forward pass's bf16 O (8 * 2^-9 ~ 0.02 absolute), which then sets the error of a row whose own
    entries are far smaller: the row-scaled check does not apply here, the tensor-wide bound and the
    Frobenius bound do."""
    Q, K, V, dO = rand_inputs(9, 1, 2, 128, 128, 64)
    mask = synth.random_mask(2, 128, 128, 0.4, seed=3)
    run_bwd(2.0 * Q, 2.0 * K, V, dO, mask, False, scale=0.2, per_row=False)


def test_backward_full_size_c5_two_slices_against_oracle():
    """The benchmark's shape and launch configuration (B4 H16 L4096 D128 causal, C5's mask); the
    gradients of two (example, head) slices are compared element by element."""
    cfg = synth.CONFIGS["C5"]
    mask = synth.make_mask(cfg)
    Q, K, V = synth.make_qkv(cfg)
    dO = np.random.default_rng([synth.SEED, 4243]).standard_normal(Q.shape, dtype=np.float32)
    dq, dk, dv, dg = (torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (Q, K, V, dO))
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64)
    lt = ap.ap_build_layout_transpose(lay)
    O, lse = ap.ap_sparse_attn_fwd(dq, dk, dv, lay, causal=True)
    gQ, gK, gV = ap.ap_sparse_attn_bwd(dq, dk, dv, O, dg, lse, lay, lt, causal=True)
    torch.cuda.synchronize()
    for t in (gQ, gK, gV):
        assert bool(torch.isfinite(t).all())
    for b, h in ((0, 0), (3, 11)):
        sl = lambda t: t[b:b + 1, h:h + 1].double().cpu().numpy()
        ref = oracle.masked_attention_backward(sl(dq), sl(dk), sl(dv), mask[h:h + 1], sl(dg), causal=True)
        for name, got, want in zip(("dQ", "dK", "dV"), (gQ, gK, gV), ref):
            print("C5 bwd", name, (b, h), assert_grad_close(name, sl(got), want, "[%d,%d]" % (b, h)), flush=True)
