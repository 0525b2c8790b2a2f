"""The native call path against the general path of the binding, over the forms of a call that it accepts and
those that it leaves alone: same outputs bit for bit, same refusals."""
import numpy as np
import pytest
import torch

from paper_2012_02030_amd import binding as ap

pytestmark = pytest.mark.gpu


class _General:
    """Stands in for the native module: every call takes the general path."""
    fwd = split = entmax_fwd = bwd = staticmethod(lambda *a: None)


def _qkv(B, H, Lq, Lk, D, dtype, strided, seed):
    g = torch.Generator().manual_seed(seed)

    def one(L):
        shape = (B, L, H, D) if strided else (B, H, L, D)
        t = torch.randn(shape, generator=g).to(dtype).cuda()
        return t.transpose(1, 2) if strided else t
    return one(Lq), one(Lk), one(Lk)


def _plan(H, Lq, Lk, causal, seed):
    rng = np.random.default_rng(seed)
    m = (rng.random((H, Lq, Lk)) < 0.3).astype(np.uint8)
    m[:, :, 0] = 1
    lay = ap.ap_build_layout(torch.from_numpy(m).cuda(), 64, 64)
    lt = ap.ap_build_layout_transpose(lay)
    return lay, ap.ap_build_schedule(lay, causal=causal), lt, ap.ap_build_col_schedule(lay, lt, causal=causal)


def _both(monkeypatch, call, native):
    ap.lib()
    seen = []

    class Watch:
        def __getattr__(self, name):
            f = getattr(real, name)

            def g(*a):
                r = f(*a)
                seen.append(r is not None)
                return r
            return g
    real = ap._calls
    with monkeypatch.context() as mp:
        mp.setattr(ap, "_calls", Watch())
        got = call()
    assert seen and all(s == native for s in seen)
    with monkeypatch.context() as mp:
        mp.setattr(ap, "_calls", _General)
        want = call()
    torch.cuda.synchronize()
    for x, y in zip(got, want):
        assert (x is None) == (y is None)
        if x is not None:
            assert x.shape == y.shape and x.stride() == y.stride() and x.dtype == y.dtype and torch.equal(x, y)
            assert not x.requires_grad


@pytest.mark.parametrize("strided", [False, True])
@pytest.mark.parametrize("causal", [False, True])
def test_native_calls_match_the_general_path(monkeypatch, causal, strided):
    B, H, Lq, Lk, D = 2, 3, 65, 97, 64
    Q, K, V = _qkv(B, H, Lq, Lk, D, torch.bfloat16, strided, 1)
    Q.requires_grad_()
    lay, sched, lt, col = _plan(H, Lq, Lk, causal, 2)
    dO = torch.randn(B, H, Lq, D, generator=torch.Generator().manual_seed(3)).to(torch.bfloat16).cuda()
    O, lse = ap.ap_sparse_attn_fwd(Q, K, V, lay, causal=causal)
    _, tau = ap.ap_sparse_attn_entmax15_fwd(Q, K, V, lay, causal=causal)
    for sc, cc in ((None, None), (sched, col), (sched, None), (None, col)):
        _both(monkeypatch, lambda: ap.ap_sparse_attn_fwd(Q, K, V, lay, causal=causal, sched=sc), True)
        _both(monkeypatch, lambda: ap.ap_sparse_attn_bwd(Q, K, V, O, dO, lse, lay, lt, causal=causal, sched=sc,
                                                         col_sched=cc), True)
    s = torch.cuda.current_stream()
    _both(monkeypatch, lambda: ap.ap_sparse_attn_fwd(Q, K, V, lay, causal=causal, return_lse=False, stream=s,
                                                     softmax_scale=0.25), True)
    _both(monkeypatch, lambda: ap.ap_sparse_attn_fwd(Q, K, V, lay, causal=causal, crop=True, sched=sched), True)
    if not causal:
        _both(monkeypatch, lambda: ap.ap_sparse_attn_fwd(Q[:, :, :50], K[:, :, :70], V[:, :, :70], lay, crop=True,
                                                         sched=sched), True)
    _both(monkeypatch, lambda: ap.ap_sparse_attn_fwd_split(Q, K, V, lay, 2, causal=causal, sched=sched), True)
    _both(monkeypatch, lambda: ap.ap_sparse_attn_decode(Q, K, V, lay, causal=causal, splits=1), True)
    _both(monkeypatch, lambda: ap.ap_sparse_attn_decode(Q, K, V, lay, causal=causal, splits=2), True)
    _both(monkeypatch, lambda: ap.ap_sparse_attn_entmax15_fwd(Q, K, V, lay, causal=causal, sched=sched), True)
    _both(monkeypatch, lambda: ap.ap_sparse_attn_entmax15_bwd(Q, K, V, dO, tau, lay, lt, sched, col, causal=causal),
          True)
    # forms that the general path keeps: dO with other strides, a log-sum-exp that is a view, other spellings of flags
    dt = dO.transpose(1, 2).contiguous().transpose(1, 2)
    _both(monkeypatch, lambda: ap.ap_sparse_attn_bwd(Q, K, V, O, dt, lse, lay, lt, causal=causal), False)
    _both(monkeypatch, lambda: ap.ap_sparse_attn_bwd(Q, K, V, O, dO, lse.transpose(0, 1).contiguous().transpose(0, 1),
                                                     lay, lt, causal=causal), False)
    _both(monkeypatch, lambda: ap.ap_sparse_attn_fwd(Q, K, V, lay, causal=int(causal)), False)
    out = torch.empty_like(O)
    _both(monkeypatch, lambda: ap.ap_sparse_attn_fwd(Q.float(), K.float(), V.float(), lay, causal=causal), True)
    assert ap.ap_sparse_attn_fwd(Q, K, V, lay, causal=causal, out=out)[0] is out


def test_refusals_are_those_of_the_general_path():
    B, H, Lq, Lk, D = 1, 2, 64, 64, 64
    Q, K, V = _qkv(B, H, Lq, Lk, D, torch.bfloat16, False, 1)
    lay, sched, lt, col = _plan(H, Lq, Lk, True, 2)
    for call in (lambda: ap.ap_sparse_attn_fwd(Q, K.float(), V, lay),
                 lambda: ap.ap_sparse_attn_fwd(Q.half(), K.half(), V.half(), lay),
                 lambda: ap.ap_sparse_attn_fwd(Q[:, :, :32], K, V, lay),
                 lambda: ap.ap_sparse_attn_fwd(Q, K, V[:, :, :32], lay),
                 lambda: ap.ap_sparse_attn_fwd(Q[0], K[0], V[0], lay),
                 lambda: ap.ap_sparse_attn_fwd(Q, K, V, lay, sched=sched),              # causal=False, schedule causal
                 lambda: ap.ap_sparse_attn_fwd(Q[..., ::2], K[..., ::2], V[..., ::2], lay),
                 lambda: ap.ap_sparse_attn_bwd(Q, K, V, Q, Q[:, :, :32], Q, lay, lt),
                 lambda: ap.ap_sparse_attn_entmax15_fwd(Q.float(), K.float(), V.float(), lay)):
        with pytest.raises(ValueError):
            call()
    with pytest.raises(ap.ApError) as e:                     # a status of the C ABI: D = 48
        ap.ap_sparse_attn_fwd(Q[..., :48].contiguous(), K[..., :48].contiguous(), V[..., :48].contiguous(), lay)
    assert e.value.status == ap.AP_ERR_UNSUPPORTED
    with pytest.raises(ap.ApError):
        ap.ap_sparse_attn_fwd_split(Q, K, V, lay, 0)


def test_transforms_and_modes_keep_to_the_general_path():
    B, H, Lq, Lk, D = 1, 2, 64, 64, 64
    Q, K, V = _qkv(B, H, Lq, Lk, D, torch.bfloat16, False, 1)
    lay = _plan(H, Lq, Lk, False, 2)[0]
    args = (Q, K, V, lay, False, 0.0, True, None, None, False)
    assert type(ap._calls.fwd(*args)) is tuple
    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode

    class F(TorchFunctionMode):
        def __torch_function__(self, func, types, a=(), k=None):
            return func(*a, **(k or {}))

    class M(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, a=(), k=None):
            return func(*a, **(k or {}))
    for mode in (F, M):
        with mode():
            assert ap._calls.fwd(*args) is None

    def under_vmap(q):
        assert ap._calls.fwd(q, K, V, lay, False, 0.0, True, None, None, False) is None
        return q
    torch.func.vmap(under_vmap)(Q[None])

    def under_grad(q):
        assert ap._calls.fwd(q, K, V, lay, False, 0.0, True, None, None, False) is None
        return q.float().sum()
    torch.func.grad(under_grad)(Q)


def test_a_side_stream_keeps_its_scratch_memory():
    """Split and backward pass on a side stream that is still busy, while the current stream goes on allocating and
    filling blocks of every size that the calls use: same results, and ready for use after one wait."""
    B, H, Lq, Lk, D = 2, 4, 128, 256, 64
    Q, K, V = _qkv(B, H, Lq, Lk, D, torch.bfloat16, False, 1)
    lay, sched, lt, col = _plan(H, Lq, Lk, True, 2)
    dO = torch.randn(B, H, Lq, D, generator=torch.Generator().manual_seed(3)).to(torch.bfloat16).cuda()
    want = ap.ap_sparse_attn_fwd_split(Q, K, V, lay, 4, causal=True, sched=sched)
    want = want + ap.ap_sparse_attn_bwd(Q, K, V, *want[:1], dO, want[1], lay, lt, causal=True, sched=sched,
                                        col_sched=col)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        busy = torch.randn(2048, 2048, device="cuda")
        for _ in range(20):
            busy = busy @ busy * 0.01
    got = ap.ap_sparse_attn_fwd_split(Q, K, V, lay, 4, causal=True, sched=sched, stream=side)
    got = got + ap.ap_sparse_attn_bwd(Q, K, V, *got[:1], dO, got[1], lay, lt, causal=True, sched=sched,
                                      col_sched=col, stream=side)
    sizes = {4 * B * H * Lq * (D + 1) * 4, B * H * Lq * 4, B * H * Lq * D * 2, B * H * Lk * D * 2}
    filled = [torch.full((n,), 255, dtype=torch.uint8, device="cuda") for n in sorted(sizes) for _ in range(4)]
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    for x, y in zip(got, want):
        assert torch.equal(x, y)
    assert all(bool((f == 255).all()) for f in filled)
