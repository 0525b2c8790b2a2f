"""GPU parity of masked attention with the 1.5-entmax normaliser (Section 6) against the fp64
oracle: O within the forward tolerance (bf16 inputs and output, P rounded to bf16 before the
second product), tau within 1e-3, and the residual |sum p - 1| at the returned tau within the
bound the header states (1e-4: Newton's iteration stops a row at a residual <= 1e-5, or one step
after a residual <= 1e-2 if that step leaves no more than 1e-4; scores are formed in fp32)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2012_02030_amd import binding as ap
from paper_2012_02030_amd import synth

from gpu_util import TOL, to_device

pytestmark = pytest.mark.gpu


def run_entmax(Q, K, V, mask, causal, scale=0.0):
    """Both walks (layout tiles, visit schedule) against the oracle."""
    dq, rq = to_device(Q, "bf16")
    dk, rk = to_device(K, "bf16")
    dv, rv = to_device(V, "bf16")
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64)
    sched = ap.ap_build_schedule(lay, causal=causal)
    O_ref, tau_ref = oracle.masked_entmax15_attention(rq, rk, rv, mask, causal=causal, scale=scale)
    err = 0.0
    for sc in (None, sched):
        O, tau = ap.ap_sparse_attn_entmax15_fwd(dq, dk, dv, lay, causal=causal, softmax_scale=scale, sched=sc)
        torch.cuda.synchronize()
        err = max(err, check_entmax(O, tau, O_ref, tau_ref))
    return err


def check_entmax(O, tau, O_ref, tau_ref):
    Oh, th = O.double().cpu().numpy(), tau.double().cpu().numpy()
    assert np.isfinite(Oh).all()
    err = float(np.abs(Oh - O_ref).max())
    assert err <= TOL["bf16"], "max |O - oracle| = %.3e" % err
    empty = np.isinf(tau_ref)
    assert np.array_equal(np.isinf(th), empty)
    if (~empty).any():
        terr = float(np.abs(th[~empty] - tau_ref[~empty]).max())
        assert terr <= 1e-3, "max |tau - oracle| = %.3e" % terr
    return err


def rand_qkv(seed, B, H, Lq, Lk, D, gain=1.0):
    rng = np.random.default_rng([synth.SEED, 1515, seed])
    return (gain * rng.standard_normal((B, H, Lq, D), dtype=np.float32),
            rng.standard_normal((B, H, Lk, D), dtype=np.float32),
            rng.standard_normal((B, H, Lk, D), dtype=np.float32))


ENTMAX_CASES = [
    # B, H, Lq, Lk, D, causal, density, query gain (sharper scores -> smaller supports)
    (2, 2, 128, 128, 64, False, 0.5, 1.0),
    (1, 2, 200, 200, 64, True, 0.3, 3.0),
    (1, 2, 100, 157, 32, False, 0.3, 1.0),
    (1, 2, 100, 300, 128, True, 0.2, 0.2),      # nearly equal scores: large supports
    (1, 1, 192, 192, 128, False, 1.0, 1.0),     # nothing pruned
    (1, 2, 64, 64, 64, True, 0.05, 1.0),        # empty rows
    (1, 1, 1, 1, 32, False, 1.0, 1.0),
]


@pytest.mark.parametrize("case", ENTMAX_CASES, ids=lambda c: "B%d_H%d_%dx%d_D%d_%s_g%g" % (c[:5] + ("causal" if c[5] else "full", c[7])))
def test_entmax_forward_matches_oracle(case):
    B, H, Lq, Lk, D, causal, density, gain = case
    Q, K, V = rand_qkv(Lq + Lk + D, B, H, Lq, Lk, D, gain)
    mask = synth.random_mask(H, Lq, Lk, density, seed=Lq + D)
    run_entmax(Q, K, V, mask, causal)


@pytest.mark.parametrize("case", ENTMAX_CASES[:5], ids=lambda c: "%dx%d_D%d_g%g" % (c[2], c[3], c[4], c[7]))
def test_entmax_returned_tau_leaves_the_documented_residual(case):
    """sum_j [x_ij - tau_i]_+^2 recomputed in fp64 from the returned tau (scores from the same
    bf16-rounded inputs) is within 1e-4 of 1 for every query with a visible kept key, for both
    walks."""
    B, H, Lq, Lk, D, causal, density, gain = case
    Q, K, V = rand_qkv(Lq + Lk + D, B, H, Lq, Lk, D, gain)
    mask = synth.random_mask(H, Lq, Lk, density, seed=Lq + D)
    dq, rq = to_device(Q, "bf16")
    dk, rk = to_device(K, "bf16")
    dv, _ = to_device(V, "bf16")
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64)
    sched = ap.ap_build_schedule(lay, causal=causal)
    keep = mask != 0
    if causal:
        keep = keep & (np.arange(Lk)[None, :] <= np.arange(Lq)[:, None] + (Lk - Lq))[None]
    x = np.einsum("bhid,bhjd->bhij", rq, rk) / (2.0 * np.sqrt(D))
    for sc in (None, sched):
        _, tau = ap.ap_sparse_attn_entmax15_fwd(dq, dk, dv, lay, causal=causal, sched=sc)
        torch.cuda.synchronize()
        th = tau.double().cpu().numpy()
        u = np.where(keep[None], np.maximum(x - th[..., None], 0.0), 0.0)
        total = (u * u).sum(-1)
        rows = keep.any(-1)[None].repeat(B, 0)
        resid = float(np.abs(total[rows] - 1.0).max())
        assert resid <= 1e-4, "max |sum p - 1| = %.3e" % resid


def test_entmax_zero_queries_give_the_mean_of_kept_values():
    Q, K, V = rand_qkv(3, 1, 2, 96, 96, 64)
    mask = synth.random_mask(2, 96, 96, 0.4, seed=8)
    run_entmax(0.0 * Q, K, V, mask, False)


def test_entmax_on_a_structured_mask_and_explicit_scale():
    cfg = synth.CONFIGS["C3"]
    mask = np.stack([synth.head_mask(cfg, h) for h in range(2)]).astype(np.uint8)
    Q, K, V = rand_qkv(5, 1, 2, cfg.Lq, cfg.Lk, cfg.D, 2.0)
    run_entmax(Q, K, V, mask, True, scale=0.2)


def test_entmax_full_size_c5_two_slices_against_oracle():
    """The benchmark's shape (B4 H16 L4096 D128 causal, C5's mask): two (example, head) slices
    element by element, and the rows of every slice are finite."""
    cfg = synth.CONFIGS["C5"]
    mask = synth.make_mask(cfg)
    Q, K, V = synth.make_qkv(cfg)
    dq, dk, dv = (torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (Q, K, V))
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64)
    sched = ap.ap_build_schedule(lay, causal=True)
    O, tau = ap.ap_sparse_attn_entmax15_fwd(dq, dk, dv, lay, causal=True, sched=sched)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(O).all()) and bool(torch.isfinite(tau).all())
    for b, h in ((0, 1), (3, 14)):
        sl = lambda t: t[b:b + 1, h:h + 1].double().cpu().numpy()
        rows = slice(0, cfg.Lq, 7)                               # every 7th query keeps the oracle quick
        O_ref, tau_ref = oracle.masked_entmax15_attention(sl(dq)[:, :, rows], sl(dk), sl(dv),
                                                          _rows_mask(mask[h:h + 1], rows, cfg), causal=False)
        assert np.abs(sl(O)[:, :, rows] - O_ref).max() <= TOL["bf16"]
        assert np.abs(sl(tau)[:, :, rows] - tau_ref).max() <= 1e-3


def _rows_mask(mask_h, rows, cfg):
    """Mask rows of the sampled queries with the causal limit folded in (the oracle is then called
    without its causal flag, which would align a query subset differently)."""
    i = np.arange(cfg.Lq)[rows][:, None]
    j = np.arange(cfg.Lk)[None, :]
    return (mask_h[:, rows, :] != 0) & (j <= i + (cfg.Lk - cfg.Lq))[None]


def test_entmax_block_row_with_more_than_64_schedule_entries():
    """Dense 64 x 5000 mask: 79 consecutive entries in the one block row, far more than are held."""
    Q, K, V = rand_qkv(11, 1, 1, 64, 5000, 64)
    mask = np.ones((1, 64, 5000), np.uint8)
    run_entmax(Q, K, V, mask, False)


def test_entmax_block_row_with_more_than_16_gathered_entries():
    """Sparse 64 x 3000 mask (2 % kept, about 45 distinct columns per tile): every tile of the one
    block row is packed, into many gathered entries; fewer with a 64 x 900 mask of the same kind."""
    for Lk, seed in ((3000, 12), (900, 13)):
        print("entmax gathered", Lk, flush=True)
        Q, K, V = rand_qkv(seed, 1, 1, 64, Lk, 64, gain=2.0)
        mask = synth.random_mask(1, 64, Lk, 0.02, seed=seed)
        lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64)
        sched = ap.ap_build_schedule(lay, causal=False)
        torch.cuda.synchronize()
        n_gathered = int((sched.start[: int(sched.cnt[0].item())] < 0).sum().item())
        assert (n_gathered > 16) == (Lk == 3000), n_gathered
        run_entmax(Q, K, V, mask, False)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("tiles", [1, 2, 3, 7, 8, 9, 10, 13])
def test_entmax_every_number_of_entries_around_those_held(tiles, D):
    """Block rows of so many entries (layout tiles; with the schedule consecutive and gathered ones), the last key
    tile and the last query tile incomplete: all held up to 8, of longer rows the first few."""
    Lk = 64 * tiles - 5
    Q, K, V = rand_qkv(tiles, 1, 2, 70, Lk, D, gain=1.5)
    mask = synth.random_mask(2, 70, Lk, 0.6, seed=tiles)
    mask[1] = synth.random_mask(1, 70, Lk, 0.02, seed=tiles)[0]        # gathered
    mask[:, 3] = 0                                                     # a query without keys
    run_entmax(Q, K, V, mask, False)


@pytest.mark.parametrize("D,kind", [(64, "equal"), (64, "ascending"), (128, "ascending"), (32, "descending"),
                                    (64, "mixed"), (128, "periodic")])
def test_entmax_start_from_the_largest_score_of_every_place(D, kind):
    """Rows whose large scores share their places in the tiles (equal, growing or periodic scores) and rows whose large
    scores do not, alone and next to each other in a block row."""
    B, H, L = 1, 2, 400
    Q, K, V = rand_qkv(D, B, H, L, L, D)
    if kind in ("ascending", "descending", "periodic"):
        along = np.linspace(-1.0, 1.0, L, dtype=np.float32) if kind != "periodic" else \
            np.where(np.arange(L) % 64 == 5, 1.0, 0.3).astype(np.float32)
        Q = np.abs(Q)
        K = (-along if kind == "descending" else along)[None, None, :, None] * np.abs(K)
    else:
        Q *= 0.0 if kind == "equal" else np.linspace(0.0, 3.0, L, dtype=np.float32)[None, None, :, None]
    mask = synth.random_mask(H, L, L, 1.0 if kind == "equal" else 0.8, seed=D)
    run_entmax(Q, K, V, mask, kind == "mixed")


# Rows in which many scores lie just above the threshold and leave the support under the last step: values of
# y = x - max x and how many keys have them.
CLUSTERED = {
    "two clusters": ((0.0, 1), (-0.999469, 1119), (-0.996444, 366), (-3.0, 50)),
    "short": ((0.0, 1), (-0.9981533752, 370), (-0.9582652282, 5)),     # 376 keys: all scores are held
    "three clusters": ((0.0, 1), (-0.998105, 3442), (-0.992293, 245), (-0.97993, 1), (-3.0, 1174)),
}


def clustered_attained_sums(names, D=32):
    """sum p at the returned tau, in 64 bits, for a query per named row (both walks).  Scores are the sum of three bf16
    parts of a key, so that the kernel's are exact to 32 bits."""
    rows = [np.repeat([v for v, _ in CLUSTERED[k]], [c for _, c in CLUSTERED[k]]) for k in names]
    y = torch.from_numpy(np.concatenate(rows))
    parts = []
    rest = y.clone()
    for _ in range(3):
        parts.append(rest.to(torch.bfloat16))
        rest = rest - parts[-1].double()
    n, Lk = len(rows), len(y)
    K = torch.zeros((1, 1, Lk, D), dtype=torch.bfloat16)
    K[0, 0, :, :3] = torch.stack(parts, 1)
    Q = torch.zeros((1, 1, n, D), dtype=torch.bfloat16)
    Q[..., :3] = 1.0
    x = K[0, 0, :, :3].double().sum(1).numpy()
    mask = np.zeros((1, n, Lk), np.uint8)
    at = 0
    for i, row in enumerate(rows):
        mask[0, i, at:at + len(row)] = 1
        at += len(row)
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64)
    sched = ap.ap_build_schedule(lay, causal=False)
    totals = []
    for sc in (None, sched):
        _, tau = ap.ap_sparse_attn_entmax15_fwd(Q.cuda(), K.cuda(), K.cuda(), lay, softmax_scale=2.0, sched=sc)
        th = tau.double().cpu().numpy()[0, 0]
        u = np.where(mask[0] != 0, np.maximum(x[None] - th[:, None], 0.0), 0.0)
        totals.append((u * u).sum(-1))
    return np.concatenate(totals)


@pytest.mark.parametrize("names", [("two clusters",), ("three clusters",), ("three clusters", "two clusters"), ("short",)])
def test_entmax_tau_never_passes_the_root(names):
    """tau rises to the root and never passes it: sum p >= 1 up to the residual 1e-5 at which a row stops (and as much
    again for the 32-bit sums over some thousand keys)."""
    assert clustered_attained_sums(names).min() >= 1.0 - 2e-5


@pytest.mark.parametrize("names", [("two clusters",), ("three clusters",), ("three clusters", "two clusters"), ("short",)])
def test_entmax_residual_where_scores_leave_the_support_under_the_last_step(names):
    """The bound of the header, |sum p - 1| <= 1e-4, on rows whose unconfirmed last step leaves 1.0e-3 and 2.4e-3."""
    total = clustered_attained_sums(names)
    assert np.abs(total - 1.0).max() <= 1e-4, total


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("Lk", [100, 300])
def test_entmax_block_rows_without_entries_are_positive_zeros(Lk, D):
    """Nobody reads the query rows of a block row that keeps nothing, and they must not reach what is written for it."""
    Q, K, V = rand_qkv(61, 4, 4, 150, Lk, D, gain=-1e30)
    mask = synth.random_mask(4, 150, Lk, 0.3, seed=62)
    mask[:, 64:128] = 0
    mask[2] = 0
    q, k, v = (to_device(x, "bf16")[0] for x in (Q, K, V))
    lay = ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64)
    for sched in (None, ap.ap_build_schedule(lay, causal=False)):
        O, tau = ap.ap_sparse_attn_entmax15_fwd(q, k, v, lay, sched=sched)
        torch.cuda.synchronize()
        assert not O[:, :, 64:128].contiguous().view(torch.int16).any() and not O[:, 2].contiguous().view(torch.int16).any()
        assert bool((tau[:, :, 64:128] == float("inf")).all()) and bool((tau[:, 2] == float("inf")).all())


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("tiles", [63, 64, 65, 66, 130])
def test_entmax_starts_of_more_entries_than_a_wavefront_has_lanes(tiles, D):
    """Block rows of 63 to 130 entries, the last of them gathered (with the schedule), odd and even numbers."""
    full = tiles - 2
    Lk = 64 * full + 1000
    Q, K, V = rand_qkv(tiles, 1, 1, 64, Lk, D, gain=1.5)
    mask = synth.random_mask(1, 64, Lk, 0.5, seed=tiles)
    mask[:, :, 64 * full:] = 0
    mask[:, 1::2, 64 * full + 7::11] = 1                               # 91 isolated keys: two gathered entries
    sched = ap.ap_build_schedule(ap.ap_build_layout(torch.from_numpy(mask).cuda(), 64, 64), causal=False)
    assert int(sched.cnt[0].item()) == tiles
    run_entmax(Q, K, V, mask, False)
