"""Timed cases of the LASAD attention path, through the calls that a program makes.

Shapes are those of ``paper_2507_01652_amd.workloads`` (head dim 64; 16 x 16, 24 x 24 and 64 x 64 token grids;
12 to 24 heads) and ragged ones between them.  A case is a dict of plain values:

  kind    "decode": one token for every sequence, through a stack of `layers` layers with a state each.
          "prefill": one layer's forward over `n` tokens from position `start`, final state kept.
          "train": one layer's forward and backward over whole sequences.
  form    "scalar" (per-head decay), "gated" (decay vector per token; `own_key`: with a key tensor of its own,
          else the tied key 1 - lambda), "layer" (activations and norm fused in), "rows" (decode only: scalar
          decay, every batch row at its own position).
  B, Hh   batch rows and heads;  H, W  token grid;  dtype  storage type of the token tensors.
"""
from __future__ import annotations

import math

import torch

from paper_2507_01652_amd import binding as lasad

D = 64                     # head dim of every model size
MOST_TOKEN_HEADS = 300_000     # a drawn prefill or training case has at most this many (the largest listed one: 393 216)


def listed():
    return [
        # One image sampled by the 12-layer, 12-head model: the smallest calls, launch and host latency.
        {"name": "decode_one_image", "kind": "decode", "form": "scalar", "B": 1, "Hh": 12, "layers": 12,
         "H": 16, "W": 16, "pos": 100, "dtype": "bf16"},
        # A small serving batch through the fused layer of the 24-layer model (activations and norm inside).
        {"name": "decode_layer_small_batch", "kind": "decode", "form": "layer", "B": 16, "Hh": 16, "layers": 24,
         "H": 24, "W": 24, "pos": 301, "dtype": "bf16"},
        # The AR-decode benchmark shape: 5120 states per layer, streamed from HBM; four of the model's layers.
        {"name": "decode_large_batch", "kind": "decode", "form": "scalar", "B": 256, "Hh": 20, "layers": 4,
         "H": 16, "W": 16, "pos": 100, "dtype": "bf16"},
        # Teacher-forced pass / prefill of the base model, 256-pixel images.
        {"name": "prefill_base", "kind": "prefill", "form": "scalar", "B": 8, "Hh": 12, "H": 16, "W": 16,
         "start": 0, "n": 256, "carry": False, "own_key": True, "dtype": "bf16"},
        # The same for the large model, 384-pixel images: the default benchmark shape.
        {"name": "prefill_large", "kind": "prefill", "form": "scalar", "B": 32, "Hh": 16, "H": 24, "W": 24,
         "start": 0, "n": 576, "carry": False, "own_key": True, "dtype": "bf16"},
        # Few, long sequences: the high-resolution grid.
        {"name": "prefill_highres", "kind": "prefill", "form": "scalar", "B": 4, "Hh": 24, "H": 64, "W": 64,
         "start": 0, "n": 4096, "carry": False, "own_key": True, "dtype": "bf16"},
        # An image continued from a kept state: mid-row start, token count that fills no tile.
        {"name": "prefill_resume_ragged", "kind": "prefill", "form": "scalar", "B": 3, "Hh": 20, "H": 24, "W": 23,
         "start": 101, "n": 311, "carry": True, "own_key": True, "dtype": "bf16"},
        # fp32 storage (1e-5 accuracy): evaluation runs and checks of a model.
        {"name": "prefill_f32", "kind": "prefill", "form": "scalar", "B": 8, "Hh": 12, "H": 16, "W": 16,
         "start": 0, "n": 256, "carry": False, "own_key": True, "dtype": "f32"},
        # The fused layer's teacher-forced pass at the benchmark shape.
        {"name": "layer_prefill_large", "kind": "prefill", "form": "layer", "B": 32, "Hh": 16, "H": 24, "W": 24,
         "start": 0, "n": 576, "carry": False, "own_key": False, "dtype": "bf16"},
        # Training with the per-head decay, large model.
        {"name": "train_scalar_large", "kind": "train", "form": "scalar", "B": 32, "Hh": 16, "H": 24, "W": 24,
         "own_key": True, "dtype": "bf16"},
        # Training the fused layer of the base model: 256 images over 8 GPUs, 256 tokens each.
        {"name": "train_layer_base", "kind": "train", "form": "layer", "B": 32, "Hh": 12, "H": 16, "W": 16,
         "own_key": False, "dtype": "bf16"},
        # Training with the vector decay on a gated layer that keeps its own key, high-resolution grid.
        {"name": "train_gated_highres", "kind": "train", "form": "gated", "B": 4, "Hh": 24, "H": 64, "W": 64,
         "own_key": True, "dtype": "bf16"},
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    Hh = rng.choice((12, 16, 20, 24))
    kind = rng.choice(("decode", "prefill", "prefill", "train"))
    if kind == "decode":
        B = _log_int(rng, 1, 256)
        H, W = rng.randint(8, 64), rng.randint(8, 64)
        layers = max(2, min(24, 20480 // (B * Hh)))           # at most as many states as decode_large_batch has
        pos = rng.randrange(1, H * W)
        if (pos + 1) % W == 0:
            pos -= 1                                    # at a row's end the decay is off: a repeated pass would pile up
        return {"kind": kind, "form": rng.choice(("scalar", "layer", "rows")), "B": B, "Hh": Hh, "layers": layers,
                "H": H, "W": W, "pos": pos, "dtype": "bf16"}
    form = rng.choice(("scalar", "gated", "layer"))
    own_key = form == "scalar" or (form == "gated" and rng.random() < 0.5)
    dtype = "f32" if rng.random() < 0.15 else "bf16"
    side = 64 if dtype == "bf16" else 32               # fp32 storage: checks and evaluation, at the smaller grids
    H, W = _log_int(rng, 8, side), _log_int(rng, 8, side)
    start = rng.randrange(0, H * W // 2) if kind == "prefill" and rng.random() < 0.4 else 0
    n = H * W - start
    if kind == "prefill" and rng.random() < 0.4:
        n = rng.randint(max(1, n // 2), n)
    room = (MOST_TOKEN_HEADS if dtype == "bf16" else MOST_TOKEN_HEADS // 4) // (Hh * n)
    B = _log_int(rng, 1, max(1, min(64, room)))
    case = {"kind": kind, "form": form, "B": B, "Hh": Hh, "H": H, "W": W, "own_key": own_key, "dtype": dtype}
    if kind == "prefill":
        case.update(start=start, n=n, carry=start > 0)
    return case


def _type(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, scale=1.0, shift=0.0):
        return torch.randn(shape, generator=gen, device="cuda").mul_(scale).add_(shift)

    dt, B, Hh = _type(case), case["B"], case["Hh"]
    gated = case["form"] in ("gated", "layer")
    if case["kind"] == "decode":
        L = case["layers"]
        s = {"case": case,
             "q": list(normal(L, B, Hh, D, scale=D ** -0.5).to(dt).unbind(0)),
             "v": list(normal(L, B, Hh, D, scale=D ** -0.5).to(dt).unbind(0)),
             "out": torch.empty((L, B, Hh, D), dtype=dt, device="cuda"),
             "state": normal(L, B, Hh, D, D, scale=0.05)}
        s["outs"], s["states"] = list(s["out"].unbind(0)), list(s["state"].unbind(0))
        if gated:
            s["z"] = list(normal(L, B, Hh, D, shift=2.0).to(dt).unbind(0))
            s["weight"] = list(normal(L, Hh, D, scale=0.1, shift=1.0).unbind(0))
        else:
            s["k"] = list(normal(L, B, Hh, D, scale=D ** -0.5).to(dt).unbind(0))
            s["gamma"] = list(torch.rand((L, Hh), generator=gen, device="cuda").mul_(0.149).add_(0.85).unbind(0))
        if case["form"] == "rows":
            # rows anywhere on the grid, none at a row's end
            row = torch.randint(0, case["H"], (B,), generator=gen, device="cuda")
            col = torch.randint(0, case["W"] - 1, (B,), generator=gen, device="cuda")
            s["pos_rows"] = (row * case["W"] + col).to(torch.int32)
        return s
    n = case["n"] if case["kind"] == "prefill" else case["H"] * case["W"]
    shape = (B, n, Hh, D)
    s = {"case": case, "q": normal(*shape, scale=D ** -0.5).to(dt), "v": normal(*shape, scale=D ** -0.5).to(dt), "k": None}
    if case["form"] == "layer":
        s["q"] = (s["q"] * D ** 0.5).to(dt)               # a pre-activation has unit variance
        s["z"] = normal(*shape, shift=2.0).to(dt)
        s["weight"] = normal(Hh, D, scale=0.1, shift=1.0)
    elif case["form"] == "gated":
        s["lam"] = torch.sigmoid(normal(*shape, shift=2.0)).to(dt)
    else:
        lo, hi = (0.90, 0.9999) if n >= 2048 else (0.85, 0.999)
        s["gamma"] = torch.rand((Hh,), generator=gen, device="cuda").mul_(hi - lo).add_(lo)
    if case["own_key"]:
        s["k"] = normal(*shape, scale=D ** -0.5).to(dt)
    if case["kind"] == "train":
        s["d_o"] = normal(*shape).to(dt)
    else:
        s["state_in"] = normal(B, Hh, D, D, scale=0.05) if case["carry"] else None
        s["state_out"] = torch.empty((B, Hh, D, D), dtype=torch.float32, device="cuda")
    return s


def _forward(s, **kw):
    c = s["case"]
    if c["form"] == "layer":
        return lasad.lasad_forward_layer(s["q"], s["z"], s["v"], c["H"], c["W"], norm_weight=s["weight"], **kw)
    if c["form"] == "gated":
        return lasad.lasad_forward_gated(s["q"], s["lam"], s["v"], c["H"], c["W"], k=s["k"], **kw)
    return lasad.lasad_forward_chunked(s["q"], s["k"], s["v"], s["gamma"], c["H"], c["W"], **kw)


def _decode(s):
    c = s["case"]
    H, W, pos = c["H"], c["W"], c["pos"]
    for i in range(c["layers"]):
        if c["form"] == "layer":
            lasad.lasad_decode_step_layer(s["q"][i], s["z"][i], s["v"][i], s["states"][i], H, W, pos,
                                          norm_weight=s["weight"][i], out=s["outs"][i])
        elif c["form"] == "rows":
            lasad.lasad_decode_step_rows(s["q"][i], s["v"][i], s["states"][i], s["pos_rows"], H, W, k=s["k"][i],
                                         gamma=s["gamma"][i], out=s["outs"][i])
        else:
            lasad.lasad_decode_step(s["q"][i], s["k"][i], s["v"][i], s["gamma"][i], s["states"][i], H, W, pos,
                                    out=s["outs"][i])
    return {"out": s["out"], "state": s["state"]}


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "decode":
        return _decode(s)
    if c["kind"] == "prefill":
        o = _forward(s, start_pos=c["start"], state_in=s["state_in"], state_out=s["state_out"])
        return {"o": o, "state": s["state_out"]}
    o = _forward(s)
    if c["form"] == "layer":
        grads = lasad.lasad_backward_layer(s["q"], s["z"], s["v"], s["d_o"], c["H"], c["W"], norm_weight=s["weight"])
    elif c["form"] == "gated":
        grads = lasad.lasad_backward_gated(s["q"], s["lam"], s["v"], s["d_o"], c["H"], c["W"], k=s["k"])
    else:
        grads = lasad.lasad_backward_chunked(s["q"], s["k"], s["v"], s["d_o"], s["gamma"], c["H"], c["W"])
    return {"o": o, "grads": list(grads)}


def work(case):
    """Bytes: every operand read once, every result written once (a decode state: both).  Operations: those of the
    recurrence, per token and head: decay, rank-one update and read-out of a D x D state (5 D^2); for the gradients
    also the adjoint state (3 D^2) and the two products with it (4 D^2), the state once more included in the first."""
    e = 2 if case["dtype"] == "bf16" else 4
    seqs = case["B"] * case["Hh"]
    if case["kind"] == "decode":
        return {"bytes": case["layers"] * seqs * (2 * 4 * D * D + 4 * e * D), "flops": case["layers"] * seqs * 5 * D * D}
    n = case["n"] if case["kind"] == "prefill" else case["H"] * case["W"]
    inputs = 4 if case["form"] == "gated" and case["own_key"] else 3
    if case["kind"] == "prefill":
        states = 2 if case["carry"] else 1
        return {"bytes": seqs * (n * (inputs + 1) * e * D + states * 4 * D * D), "flops": seqs * n * 5 * D * D}
    return {"bytes": seqs * n * (2 * inputs + 2) * e * D, "flops": seqs * n * (5 + 12) * D * D}


def tolerance(case):
    """bf16 results: four times the 1.7e-3 that separates them from the same call on fp32 storage (their rounding).
    fp32 results: four times the 5e-6 by which two summation orders of the decay gradient differ (it is a small
    difference of large sums); every other fp32 tensor differs by 3e-7 between two kernels."""
    if case["dtype"] == "bf16":
        return {"rel": 7e-3}
    return {"rel": 2e-5 if case["kind"] == "train" else 1e-5}
