"""A call with a `stream` of its own takes its outputs, its scratch memory and its copies of inputs under that stream
(CPU: the library and torch's stream functions are stand-ins that record what happens where)."""
import types

import pytest
import torch

from paper_2012_02030_amd import binding as ap

SIDE, CURRENT = 77, 5


class _Library:
    """Every call succeeds without doing anything; sizes are small numbers.  Notes the stream of every call."""

    def __init__(self, now):
        self.now, self.launched = now, []

    def __getattr__(self, name):
        if name == "ap_layout_max_tiles":
            return lambda *a: 4
        if name.endswith("_bytes"):
            return lambda *a: 64

        def call(*a):
            self.launched.append((a[-1], self.now[0]))
            return 0
        return call


class _Tensor(torch.Tensor):
    """A CPU tensor that says it is on a GPU."""
    is_cuda = True


def _cuda(t):
    return t.as_subclass(_Tensor)


def _calls():
    B, H, L, D = 1, 2, 64, 32
    q = torch.zeros(B, H, L, D, dtype=torch.bfloat16)
    rows = torch.zeros(B, H, L)
    i32 = torch.zeros(8, dtype=torch.int32)
    i64 = torch.zeros(4, 64, 1, dtype=torch.int64)
    lay = ap.Layout(i32, i32[:4], i64, i64.view(-1)[:1], H, L, L, 64, 64)
    lt = ap.LayoutT(i32, i32, i32)
    sc = ap.Schedule(i32, i32, i32, i64, False, 0)
    mask, amap = torch.ones(H, L, 2 * L, dtype=torch.uint8)[:, :, ::2], torch.zeros(H, L, 2 * L)[:, :, ::2]
    turned = q.transpose(1, 2).contiguous().transpose(1, 2)
    view = rows.transpose(1, 2).contiguous().transpose(1, 2)
    return {
        "layout": lambda s: ap.ap_build_layout(_cuda(mask), stream=s),
        "layout_from_map": lambda s: ap.ap_build_layout_from_map(_cuda(amap), torch.zeros(1), stream=s),
        "schedule": lambda s: ap.ap_build_schedule(lay, stream=s),
        "fwd": lambda s: ap.ap_sparse_attn_fwd(q, q, q, lay, stream=s),
        "decode": lambda s: ap.ap_sparse_attn_decode(q, q, q, lay, stream=s, splits=2),
        "split": lambda s: ap.ap_sparse_attn_fwd_split(q, q, q, lay, 2, stream=s),
        "entmax_fwd": lambda s: ap.ap_sparse_attn_entmax15_fwd(q, q, q, lay, stream=s),
        "transpose": lambda s: ap.ap_build_layout_transpose(lay, s),
        "col_schedule": lambda s: ap.ap_build_col_schedule(lay, lt, False, 0, s),
        "bwd": lambda s: ap.ap_sparse_attn_bwd(q, q, q, q, turned, view, lay, lt, stream=s, sched=sc),
        "entmax_bwd": lambda s: ap.ap_sparse_attn_entmax15_bwd(q, q, q, q, view, lay, lt, sc, sc, stream=s),
        "maps": lambda s: ap.ap_accumulate_attention_maps(q, q, stream=s, lse=view),
        "prune": lambda s: ap.ap_prune_mask(_cuda(amap), 0.5, stream=s),
    }


@pytest.mark.parametrize("name", sorted(_calls()))
def test_memory_of_a_call_belongs_to_the_stream_it_launches_on(monkeypatch, name):
    call = _calls()[name]
    now = [CURRENT]                                          # handle of torch's current stream
    taken = []                                               # the current stream at every allocation and copy
    lib = _Library(now)

    class Switch:
        def __init__(self, s):
            self.s = s

        def __enter__(self):
            self.back, now[0] = now[0], int(self.s.cuda_stream)

        def __exit__(self, *a):
            now[0] = self.back

    def noting(f):
        def g(*a, **k):
            taken.append(now[0])
            return f(*a, **k)
        return g
    handle = lambda h: types.SimpleNamespace(cuda_stream=h)
    monkeypatch.setattr(ap, "_lib", lib)
    monkeypatch.setattr(ap, "_calls", types.SimpleNamespace(**{k: (lambda *a: None) for k in (
        "fwd", "split", "entmax_fwd", "bwd")}))
    monkeypatch.setattr(ap, "_current_handle", lambda: now[0], raising=False)
    monkeypatch.setattr(ap, "_as_stream", lambda s: s, raising=False)
    monkeypatch.setattr(torch.cuda, "stream", Switch)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: handle(now[0]))
    for f in ("empty", "empty_strided"):
        monkeypatch.setattr(torch, f, noting(getattr(torch, f)))
    for f in ("contiguous", "clone"):
        monkeypatch.setattr(torch.Tensor, f, noting(getattr(torch.Tensor, f)))
    for stream, expect in ((handle(SIDE), SIDE), (None, CURRENT), (handle(CURRENT), CURRENT)):
        del taken[:], lib.launched[:]
        call(stream)
        assert taken and set(taken) == {expect}, taken
        assert lib.launched == [(expect, expect)]
        assert now[0] == CURRENT
