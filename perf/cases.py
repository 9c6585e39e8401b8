"""The work that a user of this library has it do, as plain cases: what to call, on which sizes, and how far two correct
implementations may differ.  Sizes are those of ``synth.CONFIGS``, ``bench.py`` and ``bench_speedup_sweep.py`` (model width
2048 split into heads of 64, 128 or 256) or generic.

    kind    "decode"     deltanet_recurrent_fwd, one or a few tokens per sequence on a kept state (generation)
            "fwd"        deltanet_fwd (inference prefill)
            "train"      deltanet_fwd_save + deltanet_bwd_saved, the training step that keeps the forward pass's tiles
            "recompute"  deltanet_fwd + deltanet_bwd, the training step that saves the memory and recomputes
    rule    "plain", "gated" (per-token decay) or "fused" (feature map, normalisation and sigmoid inside the call)
    packed  0: dense [B, L, H, d]; otherwise B sequences of random lengths up to L, laid out one after the other
    states  whether the call takes an initial state (and, backward, the gradient with respect to the final one)
"""
from __future__ import annotations

import random

import numpy as np
import torch

import paper_2406_06484_amd as dn
from paper_2406_06484_amd.binding import _shape_of
from paper_2406_06484_amd.synth import draw_lengths


def _case(kind, B, L, H, dk, dv=0, dtype="bf16", rule="plain", packed=0, states=0, name=None):
    c = dict(kind=kind, rule=rule, dtype=dtype, B=B, L=L, H=H, dk=dk, dv=dv or dk, packed=packed, states=states)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one generated token for each of 32 sequences of a 1.3B-model layer: the state is read and written once
        _case("decode", 32, 1, 16, 128, states=1, name="decode_b32"),
        # the smallest training step: a fp32 layer of two heads over one short sequence; launches and latency count
        _case("train", 1, 256, 2, 64, dtype="f32", name="step_small_f32"),
        # one prompt of an odd length continued from an earlier state: few chains, a ragged last chunk
        _case("fwd", 1, 1000, 16, 128, states=1, name="prompt_1000"),
        # prefill of a batch at the size of the 1.3B model's layers
        _case("fwd", 8, 2048, 16, 128, name="prefill_b8"),
        # the training step of such a layer (the workload of bench.py)
        _case("train", 8, 2048, 16, 128, name="train_b8"),
        # the step for users who cannot keep the tiles, on a batch of odd-sized sequences
        _case("recompute", 5, 1500, 16, 128, states=1, name="recompute_ragged"),
        # half-size heads: twice as many chains over the same width, fewer and longer sequences
        _case("train", 4, 4096, 32, 64, name="train_d64"),
        # double-size heads
        _case("train", 8, 2048, 8, 256, name="train_d256"),
        # the gated rule's training step
        _case("train", 8, 2048, 16, 128, rule="gated", name="train_gated"),
        # the training step with the layer's prologue inside the call
        _case("train", 8, 2048, 16, 128, rule="fused", name="train_fused"),
        # one long sequence with states at both ends (context-parallel or truncated backpropagation)
        _case("train", 1, 32768, 16, 128, states=1, name="train_long"),
        # a packed batch of sequences of 128 to 8192 tokens
        _case("train", 14, 8192, 16, 128, packed=65536, name="train_packed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng: random.Random):
    kind = rng.choice(["decode", "fwd", "fwd", "train", "train", "train", "recompute"])
    if kind == "decode":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        return _case("decode", _log_int(rng, 1, 96), rng.choice([1, 1, 1, 2, 3, 5]), rng.choice([4, 8, 16, 24]), rng.choice([64, 128, 128, 256]),
                     dtype=dtype, rule=rng.choice(["plain", "plain", "gated"]), states=1)
    rule = rng.choice(["plain", "plain", "plain", "gated", "fused"])
    if rng.random() < 0.12:  # fp32: the precision mode, on small layers
        dk, dv = rng.choice([(64, 64), (64, 64), (32, 64), (64, 32)])
        return _case(kind, rng.randint(1, 3), _log_int(rng, 30, 1500), rng.randint(1, 8), dk, dv, dtype="f32", rule=rule, states=rng.randint(0, 1))
    dk, dv = rng.choice([(128, 128), (128, 128), (128, 128), (64, 64), (256, 256), (64, 128), (128, 64)])
    H = rng.choice([2048 // dk, 2048 // dk, 1024 // dk, rng.randint(3, 2048 // dk)])
    states = rng.randint(0, 1)
    most = 32768 if dk < 256 and dv < 256 else 16384  # tokens
    if rng.random() < 0.25:
        total = _log_int(rng, 2000, most)
        return _case(kind, 0, min(total, _log_int(rng, 300, 8192)), H, dk, dv, rule=rule, packed=total, states=states)
    L = _log_int(rng, 60, 8192)
    return _case(kind, max(1, min(32, _log_int(rng, 300, most) // L)), L, H, dk, dv, rule=rule, states=states)


def _lengths(case):
    """Packed offsets of a case: lengths uniform in [128, L] (or [L / 2, L] for short ones), the last one cut."""
    lo = 128 if case["L"] > 128 else max(1, case["L"] // 2)
    return draw_lengths(np.random.default_rng(case["packed"] + 31 * case["L"]), case["packed"], lo, case["L"])


def _shape(case):
    """(leading dimensions of the token tensors, number of chains' states, cu_seqlens on the host or None)"""
    if case["packed"]:
        cu = _lengths(case)
        return (case["packed"],), len(cu) - 1, cu
    return (case["B"], case["L"]), case["B"], None


def prepare(case, seed):
    dev, H, dk, dv = torch.device("cuda"), case["H"], case["dk"], case["dv"]
    tdt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    lead, N, cu = _shape(case)
    g = torch.Generator(device=dev).manual_seed(seed)
    randn = lambda *s: torch.randn(s, generator=g, device=dev)
    unit = lambda: torch.nn.functional.normalize(randn(*lead, H, dk), dim=-1).to(tdt)
    fused, back = case["rule"] == "fused", case["kind"] in ("train", "recompute")
    st = dict(case=case)
    # q, k unit vectors, beta = sigmoid(N(0, 1)), v, do ~ N(0, 1); for the fused rule what the projections hand over
    st["q"], st["k"] = (randn(*lead, H, dk).to(tdt), randn(*lead, H, dk).to(tdt)) if fused else (unit(), unit())
    st["v"] = randn(*lead, H, dv).to(tdt)
    st["beta"] = randn(*lead, H).to(tdt) if fused else torch.sigmoid(randn(*lead, H)).to(tdt)
    if case["rule"] == "gated":  # alpha ~ U(0.9, 1)
        st["g"] = torch.log(0.9 + 0.1 * torch.rand((*lead, H), generator=g, device=dev))
    st["S0"] = 0.02 * randn(N, H, dk, dv) if case["states"] and case["kind"] != "decode" else None
    if case["kind"] == "decode":
        st["S0"] = 0.3 * randn(N, H, dk, dv)  # a state that many tokens have written to
    if back:
        st["d_o"] = randn(*lead, H, dv).to(tdt)
        st["dST"] = randn(N, H, dk, dv) if case["states"] else None
    st["ckw"] = {}
    if cu is not None:
        st["ckw"] = dict(cu_seqlens=torch.from_numpy(cu).to(dev), cu_seqlens_host=cu)
    # the buffers a training loop or a server keeps: the workspace (saved tiles), outputs and gradients
    if case["kind"] != "decode":
        s = _shape_of(st["q"], st["v"], st["ckw"].get("cu_seqlens"), 64, [], cu)
        size = {"plain": dn.deltanet_workspace_bytes, "gated": dn.deltanet_gated_workspace_bytes, "fused": dn.deltanet_fused_workspace_bytes}
        st["ws"] = torch.empty(size[case["rule"]](s, back), dtype=torch.uint8, device=dev)
    st["okw"] = dict(o=torch.empty_like(st["v"]), final_state=torch.empty(N, H, dk, dv, device=dev))
    if back:
        st["gkw"] = dict(dq=torch.empty_like(st["q"]), dk=torch.empty_like(st["k"]), dv=torch.empty_like(st["v"]),
                         dbeta=torch.empty(*lead, H, device=dev), dinitial_state=torch.empty(N, H, dk, dv, device=dev))
        if case["rule"] == "gated":
            st["gkw"]["dg"] = torch.empty(*lead, H, device=dev)
    return st


_CALLS = {  # (forward, forward that keeps tiles, backward, backward on kept tiles)
    "plain": (dn.deltanet_fwd, dn.deltanet_fwd_save, dn.deltanet_bwd, dn.deltanet_bwd_saved),
    "gated": (dn.deltanet_gated_fwd, dn.deltanet_gated_fwd_save, dn.deltanet_gated_bwd, dn.deltanet_gated_bwd_saved),
    "fused": (dn.deltanet_fused_fwd, dn.deltanet_fused_fwd_save, dn.deltanet_fused_bwd, dn.deltanet_fused_bwd_saved),
}


def run(st):
    case, ckw, okw = st["case"], st["ckw"], st["okw"]
    args = [st["q"], st["k"], st["v"], st["beta"]] + ([st["g"]] if case["rule"] == "gated" else [])
    if case["kind"] == "decode":
        return (dn.deltanet_gated_recurrent_fwd if case["rule"] == "gated" else dn.deltanet_recurrent_fwd)(*args, st["S0"], **okw)
    fwd, fwd_save, bwd, bwd_saved = _CALLS[case["rule"]]
    if case["kind"] == "fwd":
        return fwd(*args, st["S0"], workspace=st["ws"], **okw, **ckw)
    if case["kind"] == "train":
        o, ST, saved = fwd_save(*args, st["S0"], saved=st["ws"], **okw, **ckw)
        grads = bwd_saved(*args, st["d_o"], saved, st["dST"], **st["gkw"], **ckw)
    else:
        o, ST = fwd(*args, st["S0"], workspace=st["ws"], **okw, **ckw)
        grads = bwd(*args, st["d_o"], st["S0"], st["dST"], workspace=st["ws"], **st["gkw"], **ckw)
    return (o, ST) + tuple(grads)


def work(case):
    """Every input read once and every output written once; operations of the token recurrence (three products of the
    state with a vector per token forward, twice that backward)."""
    lead, N, _ = _shape(case)
    rows, es = case["H"] * int(np.prod(lead)), 2 if case["dtype"] == "bf16" else 4
    dk, dv, back, gated = case["dk"], case["dv"], case["kind"] in ("train", "recompute"), case["rule"] == "gated"
    state = 4 * N * case["H"] * dk * dv
    by = rows * es * (2 * dk + dv + 1 + dv) + (4 * rows if gated else 0)            # q, k, v, beta, g in; o out
    by += state * (2 if case["states"] else 1)                                      # S0 in; final state out
    fl = 6 * rows * dk * dv
    if back:
        by += rows * es * (2 * dk + dv + 1 + dv) + rows * es * (2 * dk + dv) + 4 * rows   # q, k, v, beta, do in; dq, dk, dv, dbeta out
        by += (8 * rows if gated else 0) + state * (2 if case["states"] else 1)           # g in, dg out; dST in, dS0 out
        fl += 12 * rows * dk * dv
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # four times what the outputs were seen to be off an evaluation of the same inputs in 64 bits
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}       # 1e-7 to 7e-7; largest entry 5e-6
    if case["kind"] == "decode":
        return {"rel": 7e-3, "max": 1.6e-2}     # fp32 arithmetic, o rounded to bf16 once: 1.7e-3, largest entry 4e-3
    if case["rule"] == "gated":
        return {"rel": 3e-2, "max": 0.2}        # the gate's gradient is a difference of bf16 sums: 8e-3; the other tensors as below
    return {"rel": 2e-2, "max": 0.2}            # bf16 tiles between fp32 accumulations: 2e-3 to 6e-3; largest entry 5.7e-2
