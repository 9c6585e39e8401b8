"""The chunk-local backward kernel at the rows where dbeta cannot be a quotient by beta: beta zero (masked tokens),
tiny or negative, alone, in runs across a chunk boundary, in a ragged last chunk, for every compiled head size and rule."""
import numpy as np
import pytest
import torch

import oracle
import paper_2406_06484_amd as dn
from paper_2406_06484_amd.synth import make_gate, make_inputs, make_pre_activations
from tests.gpu_util import check_fwd_bwd, dev_inputs, gpu_bwd
from tests.test_gpu_fused import run_fused
from tests.test_gpu_gated import run_gated

pytestmark = pytest.mark.gpu


def _masked(dtype, dk, dv, seed, cu=None):
    kw = dict(cu_seqlens=cu) if cu is not None else dict(B=2, L=200)
    inp = make_inputs(seed, H=2, dk=dk, dv=dv, dtype=dtype, with_initial_state=True, with_dfinal_state=True, **kw)
    b = inp.beta.reshape(-1, 2) if cu is not None else inp.beta
    tok = (lambda s: (s,)) if cu is not None else (lambda s: (slice(None), s))
    b[tok(slice(3, 4))] = 0.0          # one token
    b[tok(slice(60, 70))] = 0.0        # a run across the chunk boundary
    b[tok(slice(80, 81))] = 2.0 ** -41 # just below, just above the line between the two forms
    b[tok(slice(81, 82))] = 2.0 ** -39
    b[tok(slice(90, 95))] *= -1.0
    b[tok(slice(195, 200))] = 0.0      # in the ragged tail
    return inp


@pytest.mark.parametrize("dtype,dk,dv", [("f32", 64, 64), ("f32", 32, 64), ("f32", 64, 32), ("bf16", 64, 64), ("bf16", 64, 128),
                                         ("bf16", 128, 64), ("bf16", 128, 128), ("bf16", 256, 256)])
def test_masked_tokens(dtype, dk, dv):
    inp = _masked(dtype, dk, dv, 500 + dk + 3 * dv)
    check_fwd_bwd(inp, label="masked %s %dx%d" % (dtype, dk, dv))
    run_gated(inp, make_gate(4, inp.beta.shape, lo=0.8, hi=1.0), label="masked gated %s %dx%d" % (dtype, dk, dv))


def test_masked_tokens_packed_and_all_masked():
    cu = np.array([0, 0, 5, 69, 199, 262, 263, 263, 520], dtype=np.int32)
    check_fwd_bwd(_masked("bf16", 128, 128, 77, cu), label="masked packed")
    inp = make_inputs(78, B=1, L=130, H=3, dk=128, dv=128, dtype="bf16", with_initial_state=True, with_dfinal_state=True)
    inp.beta[:] = 0.0
    check_fwd_bwd(inp, label="all masked")


SIZES = [("f32", 64, 64), ("f32", 32, 64), ("f32", 64, 32), ("bf16", 64, 64), ("bf16", 64, 128), ("bf16", 128, 64), ("bf16", 128, 128), ("bf16", 256, 256)]


@pytest.mark.parametrize("dtype,dk,dv", SIZES)
def test_rows_of_masked_tokens_on_their_own(dtype, dk, dv):
    """The gradients of those rows alone, which a whole tensor's error would hide: exact zeros of dk and dv where beta is zero,
    and where it is tiny dk and dv of its size, held to the bound that whole tensors have (they are rows like any other)."""
    inp = _masked(dtype, dk, dv, 900 + dk + 3 * dv)
    inp.beta[:, 100] = -2.0 ** -60
    _, gk, gv, gb, _ = gpu_bwd(inp)
    _, rk, rv, rb, _ = oracle.bwd(inp.q, inp.k, inp.v, inp.beta, inp.d_o, inp.initial_state, inp.dfinal_state)
    zero, tiny = inp.beta == 0, (np.abs(inp.beta) < 2.0 ** -38) & (inp.beta != 0)
    assert zero.sum() == 2 * 2 * 16 and tiny.sum() == 2 * 2 * 3
    assert not gk[zero].any() and not gv[zero].any()
    tol = 2e-2 if dtype == "bf16" else 1e-5
    for name, x, r, rows in (("dk", gk, rk, tiny), ("dv", gv, rv, tiny), ("dbeta", gb, rb, tiny), ("dbeta", gb, rb, zero)):
        x, r = x[rows].astype(np.float64), r[rows]
        w = 1.0 / np.abs(inp.beta[rows])[:, None] if name != "dbeta" else 1.0   # (every row counts, whatever its beta)
        err = np.linalg.norm((x - r) * w) / np.linalg.norm(r * w)
        print(dtype, dk, dv, name, "%.2e" % err, flush=True)
        assert err <= tol, name


@pytest.mark.parametrize("dtype,dk,dv", SIZES)
def test_fused_rule_with_logits_far_below_zero(dtype, dk, dv):
    inp = make_pre_activations(8, make_inputs(600 + dk + dv, B=2, L=200, H=2, dk=dk, dv=dv, dtype=dtype, with_initial_state=True, with_dfinal_state=True))
    inp.beta[:, 3], inp.beta[:, 60:70], inp.beta[:, 81], inp.beta[:, 195:] = -30.0, -40.0, -120.0, -400.0
    run_fused(inp, "fused, masked %s %dx%d" % (dtype, dk, dv))
    d = dev_inputs(inp)
    gb = dn.deltanet_fused_bwd(d["q"], d["k"], d["v"], d["beta"], d["d_o"], d["S0"], d["dST"])[3].cpu().numpy()
    rb = oracle.fused_bwd(inp.q, inp.k, inp.v, inp.beta, inp.d_o, inp.initial_state, inp.dfinal_state)[3]
    assert not gb[inp.beta == -400.0].any()
    for logit in (-30.0, -40.0):
        x, r = gb[inp.beta == logit].astype(np.float64), rb[inp.beta == logit]
        assert np.linalg.norm(x - r) <= (2e-2 if dtype == "bf16" else 1e-5) * np.linalg.norm(r), logit


@pytest.mark.parametrize("rule", ["plain", "gated", "fused"])
def test_masked_tokens_cost_no_second_pass(rule):
    """A training step on a batch with a tenth of its tokens masked, and on one padded to a common length, beside the same step
    without: 1.03 to 1.08 times as long (a kernel that walked the chunks with such rows twice took 2.3 to 4.3 times)."""
    B, L, H, d = 8, 2048, 16, 128
    g = torch.Generator(device="cuda").manual_seed(1)
    randn = lambda *s: torch.randn(s, generator=g, device="cuda")
    q, k = (torch.nn.functional.normalize(randn(B, L, H, d), dim=-1).bfloat16() for _ in range(2))
    v, d_o, logit = randn(B, L, H, d).bfloat16(), randn(B, L, H, d).bfloat16(), randn(B, L, H)
    none = torch.zeros(B, L, dtype=torch.bool, device="cuda")
    tenth = torch.rand(B, L, generator=g, device="cuda") < 0.1
    padded = torch.arange(L, device="cuda")[None] >= torch.linspace(L // 2, L, B, device="cuda")[:, None]
    extra = [torch.log(0.9 + 0.1 * torch.rand(B, L, H, generator=g, device="cuda"))] if rule == "gated" else []
    pre = {"plain": "", "gated": "gated_", "fused": "fused_"}[rule]
    fwd, bwd = (getattr(dn, "deltanet_%s%s" % (pre, n)) for n in ("fwd_save", "bwd_saved"))
    best = {}
    for _ in range(3):
        for name, mask in (("none", none), ("tenth", tenth), ("padded", padded)):
            beta = torch.where(mask[..., None], torch.tensor(-200.0, device="cuda"), logit)
            beta = (beta if rule == "fused" else torch.sigmoid(beta)).bfloat16()
            assert rule == "fused" or not beta[mask].any()
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            saved = None
            for i in range(12):
                if i == 2:
                    a.record()
                o, ST, saved = fwd(q, k, v, beta, *extra, saved=saved)
                bwd(q, k, v, beta, *extra, d_o, saved)
            b.record()
            b.synchronize()
            best[name] = min(best.get(name, 1e9), a.elapsed_time(b) / 10)
    print(rule, best, flush=True)
    assert best["tenth"] <= 1.3 * best["none"] and best["padded"] <= 1.3 * best["none"]
