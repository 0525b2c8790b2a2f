"""The backward pass of short sequences (one launch for dQ, dK and dV) against the fp64 oracle, and against the kernels
of longer ones on the same problem with more queries and keys that nobody keeps."""
import numpy as np
import pytest
import torch

from paper_2012_02030_amd import binding as ap
from paper_2012_02030_amd import synth

from test_gpu_bwd import run_bwd
from test_gpu_bwd_sched import nan_padded

pytestmark = pytest.mark.gpu

# around the edges of 32-row blocks, of 64-row tiles and of the kernel's sizes, and where few keys per query or few
# pairs send a call to the general kernels
SIZES = [(1, 1), (31, 33), (33, 31), (64, 64), (65, 64), (64, 65), (127, 129), (128, 256), (129, 96), (100, 20), (40, 256)]


def rand(seed, B, H, L, D):
    return np.random.default_rng([synth.SEED, 77, seed]).standard_normal((B, H, L, D), dtype=np.float32)


@pytest.mark.parametrize("D", [32, 64])
@pytest.mark.parametrize("Lq,Lk", SIZES)
def test_short_backward_matches_oracle(Lq, Lk, D):
    B, H = 2, 3
    for causal in ((False, True) if Lk >= Lq else (False,)):
        print(Lq, Lk, D, causal, flush=True)
        mask = synth.random_mask(H, Lq, Lk, 0.4, seed=Lq + Lk)
        mask[1, :, : Lk // 2] = 0                                      # empty tiles, queries without keys
        mask[2] = Lq < 65                                              # everything, or nothing at all
        run_bwd(rand(1, B, H, Lq, D), rand(2, B, H, Lk, D), rand(3, B, H, Lk, D), rand(4, B, H, Lq, D), mask, causal)


def strided(x):
    """The same values as a view of a [B, L, H, D] tensor."""
    return x.transpose(1, 2).contiguous().transpose(1, 2)


@pytest.mark.parametrize("form", [lambda x: x, strided], ids=["contiguous", "strided"])
@pytest.mark.parametrize("B,H,Lq,Lk,D", [(2, 2, 100, 70, 64), (3, 1, 128, 250, 32), (24, 8, 256, 255, 64),
                                         (24, 8, 130, 256, 32), (24, 8, 200, 97, 64)])
def test_short_backward_matches_the_kernels_of_longer_sequences(B, H, Lq, Lk, D, form):
    """From the same O and lse, P and dS are formed and rounded to bf16 alike in all of them; sums in 32 bits in another
    order (delta, the results) turn a rounding where a value lies next to the middle of two: a unit in the last place
    of a result (2^-7 of it at most) and 2^-8 of a term of its sum, which is no larger than the largest results."""
    L = 320
    g = torch.Generator().manual_seed(Lq * 7 + Lk)
    Q, dO = (torch.randn(B, H, L, D, generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    K, V = (torch.randn(B, H, L, D, generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    mask = np.zeros((H, L, L), np.uint8)
    mask[:, :Lq, :Lk] = synth.random_mask(H, Lq, Lk, 0.2, seed=Lk)
    whole = torch.from_numpy(mask).cuda()
    lay = ap.ap_build_layout(whole, 64, 64)
    lay_t = ap.ap_build_layout_transpose(lay)
    want = []
    O, lse = ap.ap_sparse_attn_fwd(Q, K, V, lay)
    for few in (None, 1, 65):                                          # tiles; all runs of 64; all gathered
        rs = None if few is None else ap.ap_build_schedule(lay, causal=False, min_cols=few)
        cs = None if few is None else ap.ap_build_col_schedule(lay, lay_t, causal=False, min_rows=few)
        grads = ap.ap_sparse_attn_bwd(Q, K, V, O, dO, lse, lay, lay_t, sched=rs, col_sched=cs)
        want.append([x[:, :, :n].double() for x, n in zip(grads, (Lq, Lk, Lk))])
    cut = [form(x[:, :, :n]) for x, n in ((Q, Lq), (K, Lk), (V, Lk), (O, Lq), (dO, Lq))]
    lse_cut = lse[:, :, :Lq].contiguous()
    small = ap.ap_build_layout(whole[:, :Lq, :Lk].contiguous(), 64, 64)
    got = ap.ap_sparse_attn_bwd(*cut, lse_cut, small, ap.ap_build_layout_transpose(small))
    torch.cuda.synchronize()
    for name, x, refs in zip(("dQ", "dK", "dV"), got, zip(*want)):
        for ref in refs:
            excess = ((x.double() - ref).abs() - ref.abs() / 128 - ref.abs().max() / 256).max()
            assert float(excess) <= 0, (name, float(excess))


@pytest.mark.parametrize("B,H,L,D", [(2, 2, 128, 64), (2, 2, 128, 32), (24, 8, 256, 64), (2, 2, 320, 64)])
def test_tiles_that_nobody_keeps_are_never_used(B, H, L, D):
    """Rows of 64 keys and of 64 queries that are not in the layout at all (padding that nobody has written, here NaN) reach
    no gradient, neither in the short kernel nor (320) in the general ones."""
    Q, K, V, dO = (rand(i, B, H, L, D) for i in range(4))
    mask = synth.random_mask(H, L, L, 0.3, seed=L + D)
    mask[:, :, 64:128] = 0
    mask[:, :64] = 0
    q, k, v, g = (torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (Q, K, V, dO))
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64)
    lt = ap.ap_build_layout_transpose(lay)

    def grads():
        O, lse = ap.ap_sparse_attn_fwd(q, k, v, lay)
        got = ap.ap_sparse_attn_bwd(q, k, v, O, g, lse, lay, lt)
        torch.cuda.synchronize()
        return got

    want = grads()
    k[:, :, 64:128] = v[:, :, 64:128] = float("nan")
    q[:, :, :64] = g[:, :, :64] = float("nan")
    for a, b in zip(grads(), want):
        assert torch.equal(a, b)                                       # (NaN equals nothing)
    assert not want[0][:, :, :64].any() and not want[1][:, :, 64:128].any() and not want[2][:, :, 64:128].any()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D", [32, 64])
@pytest.mark.parametrize("B,H,Lq,Lk", [(2, 2, 50, 60), (1, 1, 91, 91), (2, 2, 128, 128), (24, 8, 200, 230)])
def test_keys_that_nobody_keeps_are_never_used(B, H, Lq, Lk, D, causal):
    """Single keys that no query keeps and single queries that keep nothing, inside tiles of the layout, with schedules that do
    not hold them: whatever stands there (NaN, infinity) changes no bit of a gradient."""
    Q, K, V, dO = (rand(20 + i, B, H, L, D) for i, L in enumerate((Lq, Lk, Lk, Lq)))
    mask = synth.random_mask(H, Lq, Lk, 0.1, seed=Lq + D)
    mask[:, np.arange(Lq), np.arange(Lq) % Lk] = 1
    keys, queries = [0, 7, 33, Lk - 1], [0, 5, 40, Lq - 1]
    mask[:, :, keys] = 0
    mask[:, queries] = 0
    q, k, v, g = (torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (Q, K, V, dO))
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64)
    lt = ap.ap_build_layout_transpose(lay)
    sched, cs = ap.ap_build_schedule(lay, causal=causal), ap.ap_build_col_schedule(lay, lt, causal=causal)

    def grads():
        got = ap.ap_sparse_attn_bwd(q, k, v, O, g, lse, lay, lt, causal=causal, sched=sched, col_sched=cs)
        torch.cuda.synchronize()
        return got

    O, lse = ap.ap_sparse_attn_fwd(q, k, v, lay, causal=causal, sched=sched)
    want = grads()
    for x, rows in ((k, keys), (v, keys), (q, queries), (g, queries)):
        x[:, :, rows] = float("nan")
    v[:, :, keys[1]] = float("inf")
    for a, b in zip(grads(), want):
        assert torch.equal(a, b)                                       # (NaN equals nothing)
    assert not want[0][:, :, queries].any() and not want[1][:, :, keys].any() and not want[2][:, :, keys].any()


@pytest.mark.parametrize("D", [32, 64])
@pytest.mark.parametrize("B,H,Lq,Lk", [(2, 2, 50, 40), (2, 2, 100, 97), (24, 8, 200, 230)])
def test_rows_behind_the_last_row_are_never_used(B, H, Lq, Lk, D):
    """In all three forms: NaN behind row L - 1 of Q, K, V, O and dO changes no bit of a gradient."""
    q, k, v, g = (torch.from_numpy(rand(9 + i, B, H, L, D)).to(torch.bfloat16).cuda()
                  for i, L in enumerate((Lq, Lk, Lk, Lq)))
    mask = synth.random_mask(H, Lq, Lk, 0.4, seed=Lq)
    mask[:, :, Lk - 1] = 1
    mask[:, Lq - 1, :] = 1
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64)
    lt = ap.ap_build_layout_transpose(lay)
    O, lse = ap.ap_sparse_attn_fwd(q, k, v, lay)
    want = ap.ap_sparse_attn_bwd(q, k, v, O, g, lse, lay, lt)
    got = ap.ap_sparse_attn_bwd(*(nan_padded(x) for x in (q, k, v, O, g)), lse, lay, lt)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)                                       # (NaN equals nothing)
