"""Performance cases of the masked-attention library: what its users have it do, as plain calls.

A case is a dict of plain values.  `prepare` makes what a program holds before the call (inputs on
the GPU, and the layout and schedules of a fixed mask, which are built once per layer), `run` makes
one pass through the public entry points of `paper_2012_02030_amd.binding`, `work` states the bytes
and operations the pass cannot do without, `tolerance` how far another correct implementation at
the same precision may be away.

Kinds of pass (`"kind"`):
  forward   ap_sparse_attn_fwd: inference, or the forward half of a step
  crop      the same under the top-left corner of a fixed mask (batches of shorter sequences)
  train     forward and backward of one layer
  backward  the backward pass alone, from a forward pass's O and log-sum-exp
  entmax    forward and backward with the 1.5-entmax normaliser
  maps      mean attention maps of a layer over two batches (before pruning)
  prune     mean maps -> threshold, mask, layout, schedules, first forward pass under them
  segment   a short segment against a long memory plus itself, split over the keys
  decode    one query or a few per head against a long memory

Masks have the structure the method finds: a band next to the diagonal, an attention sink, rare
long-range connections, kept by rank per head (`synth.py` describes it); they are drawn here on the
GPU, from the seed alone.
"""
import math

import torch

from paper_2012_02030_amd import binding as ap


def listed():
    return [
        # the smallest call there is: two heads of 64 queries in fp32 (unit-test and toy-model size);
        # launches and host work are all of it
        dict(name="forward_tiny_f32", kind="forward", B=1, H=2, Lq=64, Lk=64, D=32, dtype="f32", causal=True,
             keep=0.10, strided=False),
        # fp32 at an ordinary size (evaluation in full precision), a length that is no multiple of anything
        dict(name="forward_lm_f32", kind="forward", B=8, H=8, Lq=500, Lk=500, D=64, dtype="f32", causal=True,
             keep=0.10, strided=False),
        # an encoder with its 128-token mask, serving a batch whose longest sentence has 101 tokens
        dict(name="crop_encoder", kind="crop", B=32, H=12, Lq=101, Lk=101, L_mask=128, D=64, dtype="bf16",
             causal=False, keep=0.50, strided=True),
        # long-context language model, the largest ordinary forward pass
        dict(name="forward_lm_long", kind="forward", B=4, H=16, Lq=4096, Lk=4096, D=128, dtype="bf16", causal=True,
             keep=0.10, strided=False),
        # training step of the cross attention of a translation model, ragged source and target
        dict(name="train_cross", kind="train", B=32, H=8, Lq=117, Lk=141, D=64, dtype="bf16", causal=False,
             keep=0.50, strided=False),
        # training step of a small language model, heads as views of the projections
        dict(name="train_lm", kind="train", B=16, H=12, Lq=512, Lk=512, D=64, dtype="bf16", causal=True, keep=0.10,
             strided=True),
        # backward pass of the long-context model
        dict(name="backward_lm_long", kind="backward", B=4, H=16, Lq=4096, Lk=4096, D=128, dtype="bf16", causal=True,
             keep=0.10, strided=False),
        # the same kind of model trained with 1.5-entmax in place of softmax
        dict(name="entmax_lm", kind="entmax", B=4, H=16, Lq=2048, Lk=2048, D=128, dtype="bf16", causal=True,
             keep=0.10, strided=False),
        # collecting a layer's mean attention maps over a data set: two batches of it
        dict(name="maps_lm", kind="maps", B=4, H=16, Lq=2048, Lk=2048, D=128, dtype="bf16", causal=True, keep=1.0,
             strided=False),
        # pruning a layer: from its mean maps to everything that its later passes need, and the first of them
        dict(name="prune_lm_long", kind="prune", B=1, H=16, Lq=4096, Lk=4096, D=128, dtype="bf16", causal=True,
             keep=0.10, strided=False),
        # a 64-token segment that attends to a cached memory of 16 thousand positions and itself
        dict(name="segment_memory", kind="segment", B=4, H=16, Lq=64, Lk=16384, D=128, dtype="bf16", causal=True,
             keep=0.10, splits=8, strided=False),
        # generation, one position at a time, against the same kind of memory (an odd number of keys)
        dict(name="decode_memory", kind="decode", B=4, H=16, Lq=1, Lk=16001, D=128, dtype="bf16", causal=True,
             keep=0.10, splits=4, strided=False),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _odd_or_round(rng, v, step):
    """Half of the drawn sizes are the multiples of `step` that programs like, the others anything."""
    return max(step, v // step * step) if rng.random() < 0.5 and v >= step else v


def draw(rng):
    kind = rng.choice(["forward_f32", "forward", "crop", "train", "train", "backward", "entmax", "maps", "prune",
                       "segment", "decode"])
    c = dict(kind=kind, dtype="bf16", causal=rng.random() < 0.7, keep=round(rng.uniform(0.08, 0.5), 3),
             strided=rng.random() < 0.5)
    D = rng.choice([64, 64, 128])
    H = rng.choice([2, 4, 6, 8, 12, 16])
    if kind == "forward_f32":
        c.update(kind="forward", dtype="f32")
        D = rng.choice([32, 64, 64, 128])
        L = _odd_or_round(rng, _log_int(rng, 16, 1024), 16)
        most = 1 << 24                                       # B * H * Lq * Lk
    elif kind in ("segment", "decode"):
        Lq = _log_int(rng, 17, 100) if kind == "segment" else rng.choice([1, 1, 2, 4])
        Lk = _odd_or_round(rng, _log_int(rng, 1024, 16384), 64)
        B = rng.randint(1, 4)
        c.update(causal=True, keep=round(rng.uniform(0.05, 0.2), 3), splits=rng.choice([2, 4, 8]), B=B, H=H, Lq=Lq,
                 Lk=Lk, D=D)
        return c
    elif kind == "crop":
        L_mask = _odd_or_round(rng, _log_int(rng, 64, 2048), 64)
        L = max(16, int(L_mask * rng.uniform(0.4, 0.98)))
        c.update(L_mask=L_mask)
        most = 1 << 27
    else:
        L = _odd_or_round(rng, _log_int(rng, 64, 2048 if kind in ("maps", "entmax") else 4096), 64)
        most = (1 << 27) if kind in ("maps", "entmax") else (1 << 29)
    Lq = Lk = L
    if kind in ("train", "forward") and not c["causal"]:     # cross attention
        Lk = max(16, int(L * rng.uniform(0.7, 1.4)))
    if not c["causal"] and c["keep"] < 0.2:
        c["keep"] = round(c["keep"] + 0.2, 3)
    if L > 1024 and kind != "maps":
        c["keep"] = min(c["keep"], 0.12)
    B = max(1, min(_log_int(rng, 1, 32), most // (H * Lq * Lk)))
    if kind == "prune":
        B = 1
    c.update(B=B, H=H, Lq=Lq, Lk=Lk, D=D)
    return c


# ---- inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _tensor(c, L, g):
    """Standard-normal [B, H, L, D]; strided: a view of a [B, L, H, D] projection."""
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    shape = (c["B"], L, c["H"], c["D"]) if c["strided"] else (c["B"], c["H"], L, c["D"])
    t = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(dt)
    return t.transpose(1, 2) if c["strided"] else t


def _score(Lq, Lk, causal, width, g):
    """A stand-in for one head's mean map [Lq, Lk] (its order, not its values, makes the mask)."""
    i = torch.arange(Lq, device="cuda", dtype=torch.float32)[:, None]
    j = torch.arange(Lk, device="cuda", dtype=torch.float32)[None, :]
    if causal:
        d = i + float(Lk - Lq) - j
        base = torch.where((d >= 0) & (d < width), 1.0 - d / width, torch.zeros((), device="cuda"))
        base = base + 0.1 / (1.0 + d.clamp(min=0.0) / width) + (j == 0)
        noise = torch.randn((Lq, Lk), generator=g, device="cuda", dtype=torch.float32)
        spikes = torch.rand((Lq, Lk), generator=g, device="cuda", dtype=torch.float32) < 0.13 / width
        return base * torch.exp(0.1 * noise) + 5.0 * spikes
    centre = i * (Lk / Lq)
    noise = torch.randn((Lq, Lk), generator=g, device="cuda", dtype=torch.float32)
    return 4.0 * ((j - centre).abs() <= 5.0) + 4.0 * ((j == 0) | (j == Lk - 1)) + torch.exp(noise)


def _visible(Lq, Lk, causal):
    return Lq * Lk - Lq * (Lq - 1) // 2 if causal else Lq * Lk


def _width(Lk):
    return max(4.0, min(128.0, Lk / 16.0))


def _mask(H, Lq, Lk, causal, keep, g):
    """uint8 [H, Lq, Lk]: the strongest `keep` of every head's visible entries, and the nearest key of every query."""
    out = torch.empty((H, Lq, Lk), dtype=torch.uint8, device="cuda")
    i = torch.arange(Lq, device="cuda")[:, None]
    j = torch.arange(Lk, device="cuda")[None, :]
    hidden = (j > i + (Lk - Lq)) if causal else None
    near = (j == i + (Lk - Lq)) if causal else (j == i * Lk // Lq)
    k = max(1, int(round(keep * _visible(Lq, Lk, causal))))
    for h in range(H):
        s = _score(Lq, Lk, causal, _width(Lk), g)
        if causal:
            s.masked_fill_(hidden, -1.0)
        limit = torch.kthvalue(s.flatten(), Lq * Lk - k + 1).values
        m = (s >= limit) | near
        out[h] = m & ~hidden if causal else m
    return out


def _plan(c, mask, backward):
    """What a program keeps of a fixed mask: layout, visit schedule, and their transposes for the backward pass."""
    p = {"layout": ap.ap_build_layout(mask, 64, 64)}
    p["sched"] = ap.ap_build_schedule(p["layout"], causal=c["causal"]) if c["dtype"] == "bf16" else None
    if backward:
        p["layout_t"] = ap.ap_build_layout_transpose(p["layout"])
        p["col_sched"] = ap.ap_build_col_schedule(p["layout"], p["layout_t"], causal=c["causal"])
    return p


def prepare(case, seed):
    c = case
    g = _gen(seed)
    s = {"c": c, "Q": _tensor(c, c["Lq"], g), "K": _tensor(c, c["Lk"], g)}
    if c["kind"] == "maps":
        s["Q2"], s["K2"] = _tensor(c, c["Lq"], g), _tensor(c, c["Lk"], g)
        return s
    s["V"] = _tensor(c, c["Lk"], g)
    if c["kind"] == "prune":
        s["abar"] = torch.stack([_score(c["Lq"], c["Lk"], c["causal"], _width(c["Lk"]), g) for _ in range(c["H"])])
        return s
    Lq_m, Lk_m = (c["L_mask"], c["L_mask"]) if c["kind"] == "crop" else (c["Lq"], c["Lk"])
    backward = c["kind"] in ("train", "backward", "entmax")
    mask = _mask(c["H"], Lq_m, Lk_m, c["causal"], c["keep"], g)
    s["plan"] = _plan(c, mask, backward)
    if c["kind"] == "decode":
        s["plan"]["sched"] = None                            # the one-query kernel walks the layout
    if backward:
        s["dO"] = torch.randn((c["B"], c["H"], c["Lq"], c["D"]), generator=g, device="cuda",
                              dtype=torch.float32).to(torch.bfloat16)
    if c["kind"] == "backward":
        s["O"], s["lse"] = ap.ap_sparse_attn_fwd(s["Q"], s["K"], s["V"], s["plan"]["layout"], causal=c["causal"],
                                                 sched=s["plan"]["sched"])
    return s


# ---- one pass

def run(state):
    s, c = state, state["c"]
    kind, causal = c["kind"], c["causal"]
    if kind == "maps":
        w = 1.0 / (2 * c["B"])
        abar = ap.ap_accumulate_attention_maps(s["Q"], s["K"], causal=causal, weight=w)
        return ap.ap_accumulate_attention_maps(s["Q2"], s["K2"], abar, causal=causal, weight=w)
    if kind == "prune":
        mask, tau = ap.ap_prune_mask(s["abar"], 1.0 - c["keep"], causal=causal)
        p = _plan(c, mask, backward=True)
        O, lse = ap.ap_sparse_attn_fwd(s["Q"], s["K"], s["V"], p["layout"], causal=causal, sched=p["sched"])
        return {"mask": mask, "tau": tau, "row_ptr": p["layout"].row_ptr, "nnz": p["layout"].nnz,
                "col_ptr": p["layout_t"].col_ptr, "O": O, "lse": lse}
    p = s["plan"]
    if kind == "decode":
        return ap.ap_sparse_attn_decode(s["Q"], s["K"], s["V"], p["layout"], causal=causal, splits=c["splits"])
    if kind == "segment":
        return ap.ap_sparse_attn_fwd_split(s["Q"], s["K"], s["V"], p["layout"], c["splits"], causal=causal,
                                           sched=p["sched"])
    if kind == "entmax":
        O, tau = ap.ap_sparse_attn_entmax15_fwd(s["Q"], s["K"], s["V"], p["layout"], causal=causal, sched=p["sched"])
        grads = ap.ap_sparse_attn_entmax15_bwd(s["Q"], s["K"], s["V"], s["dO"], tau, p["layout"], p["layout_t"],
                                               p["sched"], p["col_sched"], causal=causal)
        return (O, tau) + tuple(grads)
    if kind == "backward":
        return ap.ap_sparse_attn_bwd(s["Q"], s["K"], s["V"], s["O"], s["dO"], s["lse"], p["layout"], p["layout_t"],
                                     causal=causal, sched=p["sched"], col_sched=p["col_sched"])
    O, lse = ap.ap_sparse_attn_fwd(s["Q"], s["K"], s["V"], p["layout"], causal=causal, sched=p["sched"],
                                   crop=kind == "crop")
    if kind != "train":
        return O, lse
    grads = ap.ap_sparse_attn_bwd(s["Q"], s["K"], s["V"], O, s["dO"], lse, p["layout"], p["layout_t"], causal=causal,
                                  sched=p["sched"], col_sched=p["col_sched"])
    return (O, lse) + tuple(grads)


# ---- what a pass cannot do without

def work(case):
    c = case
    B, H, Lq, Lk, D = c["B"], c["H"], c["Lq"], c["Lk"], c["D"]
    size = 4 if c["dtype"] == "f32" else 2
    q, k, rows = size * B * H * Lq * D, size * B * H * Lk * D, 4 * B * H * Lq
    pattern = H * Lq * Lk // 8                               # one bit per entry says what is kept
    visible = _visible(Lq, Lk, c["causal"])
    kept = c["keep"] * visible * B * H                       # connections of the pass
    if c["kind"] == "maps":                                  # scores once; the map written once
        return {"bytes": 2 * (q + k) + 4 * H * visible, "flops": 2 * 2 * D * visible * B * H}
    if c["kind"] == "prune":                                 # the maps once, the mask once, a forward pass
        return {"bytes": 4 * H * visible + H * Lq * Lk + pattern + 2 * q + 2 * k + rows, "flops": 4 * D * kept}
    if c["kind"] in ("segment", "decode"):                   # only rows that some query keeps are read
        far = 1.0 - (1.0 - 0.13 / _width(Lk)) ** (Lq - 1)    # isolated connections of the other queries
        used = min(1.0, c["keep"] + (1.0 - c["keep"]) * far + (Lq - 1) / Lk)
        return {"bytes": 2 * q + 2 * k * used + pattern + rows, "flops": 4 * D * kept}
    forward, backward = 4 * D * kept, 10 * D * kept
    if c["kind"] == "backward":                              # Q, K, V, O, dO, lse in; dQ, dK, dV out
        return {"bytes": 4 * q + 4 * k + rows + pattern, "flops": backward}
    if c["kind"] in ("train", "entmax"):                     # Q, K, V, dO in; O, lse, dQ, dK, dV out
        return {"bytes": 4 * q + 4 * k + rows + pattern, "flops": forward + backward}
    return {"bytes": 2 * q + 2 * k + rows + pattern, "flops": forward}


def tolerance(case):
    # Each figure is about four times what the path showed against the same result in 64 bits
    # (rel 2.1e-3 to 2.5e-3 in bf16, 1.3e-7 for fp32 attention, 2.9e-7 for the maps), with room for
    # the rows and sums that are longer than those.
    if case["kind"] == "maps":                               # 32-bit scores and hardware exponentials
        return {"rel": 2e-6, "max": 3e-5}
    if case["dtype"] == "f32":                               # 32-bit products, sums and exponentials
        return {"rel": 1e-6, "max": 1e-5}
    # bf16 results, probabilities rounded to bf16 before the second product; masks, pointers and
    # counts are whole numbers and do not differ at all
    return {"rel": 1e-2, "max": 0.2, "differ": 0.0}
