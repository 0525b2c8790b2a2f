"""GPU parity of ap_sparse_attn_decode (a few queries against many keys, Section 4.1's cached
memory taken to its limit) against the fp64 oracle, to the forward tolerance (2e-2 for bf16)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2012_02030_amd import binding as ap
from paper_2012_02030_amd import synth

from gpu_util import TOL, to_device

pytestmark = pytest.mark.gpu


def run_decode(B, H, Lq, Lk, D, causal, mask, seed, scale=0.0, block_m=64, splits=1):
    rng = np.random.default_rng([synth.SEED, 515, seed])
    Q, K, V = (rng.standard_normal(s, dtype=np.float32) for s in ((B, H, Lq, D), (B, H, Lk, D), (B, H, Lk, D)))
    dq, rq = to_device(Q, "bf16")
    dk, rk = to_device(K, "bf16")
    dv, rv = to_device(V, "bf16")
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), block_m, 64)
    print("decode", B, H, Lq, Lk, D, causal, flush=True)
    O, lse = ap.ap_sparse_attn_decode(dq, dk, dv, lay, causal=causal, softmax_scale=scale, splits=splits)
    torch.cuda.synchronize()
    O_ref, lse_ref = oracle.masked_attention(rq, rk, rv, mask, causal=causal, scale=scale)
    O_h, lse_h = O.double().cpu().numpy(), lse.double().cpu().numpy()
    assert np.isfinite(O_h).all()
    assert np.abs(O_h - O_ref).max() <= TOL["bf16"]
    empty = np.isneginf(lse_ref)
    assert np.array_equal(np.isneginf(lse_h), empty)
    if (~empty).any():
        assert np.abs(lse_h[~empty] - lse_ref[~empty]).max() <= TOL["bf16"]
    return O, lse, (dq, dk, dv, lay)


@pytest.mark.parametrize("shape", [
    (2, 3, 1, 1000, 128, True, 0.1),
    (1, 2, 3, 4099, 64, True, 0.02),       # ragged key count, a few queries
    (2, 2, 16, 700, 32, False, 0.3),
    (1, 2, 1, 1, 64, False, 1.0),
    (1, 1, 5, 300, 128, True, 1.0),        # nothing pruned
    (1, 3, 70, 200, 64, True, 0.05),       # more queries than a tile holds: still correct
])
@pytest.mark.parametrize("splits", [1, 3, 8])
def test_decode_matches_oracle(shape, splits):
    B, H, Lq, Lk, D, causal, density = shape
    mask = synth.random_mask(H, Lq, Lk, density, seed=Lk + D)
    run_decode(B, H, Lq, Lk, D, causal, mask, seed=Lk, splits=splits)


def test_decode_empty_rows_large_scores_and_wide_blocks():
    H, Lq, Lk, D = 2, 4, 500, 64
    mask = synth.random_mask(H, Lq, Lk, 0.2, seed=3)
    mask[0, 1] = 0                                     # a query without kept keys
    mask[1, :, :] = 0
    mask[1, 2, 499] = 1                                # a single kept key: O is that value row
    for splits in (1, 4):
        O, _, (dq, dk, dv, _) = run_decode(2, H, Lq, Lk, D, False, mask, seed=1, scale=0.7, splits=splits)
        assert torch.equal(O[:, 1, 2], dv[:, 1, 499])
        assert bool((O[:, 0, 1] == 0).all())
    run_decode(1, H, Lq, Lk, D, False, mask, seed=2, block_m=128, splits=2)


def test_decode_agrees_with_the_tiled_kernel_on_the_long_memory_shape():
    """X1's mask (16 heads, 64 queries, 16384 keys, causal bottom-right): its last query as a
    one-query call, against the oracle and against ap_sparse_attn_fwd's last row."""
    cfg = synth.EXTRA_CONFIGS["X1"]
    full = synth.make_mask(cfg)
    mask = np.ascontiguousarray(full[:, -1:, :])       # causal with Lq = 1: everything is visible
    O, lse, (dq, dk, dv, lay) = run_decode(2, cfg.H, 1, cfg.Lk, cfg.D, True, mask, seed=7, splits=8)
    O2, lse2 = ap.ap_sparse_attn_fwd(dq, dk, dv, lay, causal=True)
    torch.cuda.synchronize()
    assert float((O.float() - O2.float()).abs().max()) <= 2e-2
    assert float((lse - lse2).abs().max()) <= 1e-3


@pytest.mark.parametrize("splits", [1, 2, 5])
def test_decode_of_more_tiles_than_one_pass_takes(splits):
    """313 stored tiles: several passes over the key list, tiles dealt over the splits, the last tile ragged."""
    mask = synth.random_mask(1, 2, 20001, 0.05, seed=9)
    run_decode(1, 1, 2, 20001, 64, True, mask, seed=9, splits=splits)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("keys", [1, 3, 4, 5, 63, 64, 65, 448, 449, 511, 512, 513, 1023, 1024, 1025, 1600])
def test_decode_of_lists_around_whole_steps_and_batches(D, keys):
    """A list of exactly so many kept keys: around one key of every stream of a wavefront (8 or 4 streams), of all
    streams (128 or 64), and around whole batches of eight per stream (1024 or 512)."""
    mask = np.zeros((1, 1, 1700), np.uint8)
    mask[0, 0, np.random.default_rng(keys).permutation(1700)[:keys]] = 1
    run_decode(1, 1, 1, 1700, D, False, mask, seed=keys)
