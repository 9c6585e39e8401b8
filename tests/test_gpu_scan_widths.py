"""The scans give 16, 32 or 64 state columns to a workgroup, by the number of chains.  The columns are independent, so copies of one
sequence, few or many, have to give the bits of the sequence alone, at the lengths where a chunk step can go wrong (one token, one
chunk less one token, one chunk, one more); the sequence alone is checked against the oracle."""
import pytest
import torch

import paper_2406_06484_amd as dn
from paper_2406_06484_amd.synth import make_gate, make_inputs, make_pre_activations
from tests.gpu_util import check_fwd_bwd, dev_inputs
from tests.test_gpu_fused import run_fused
from tests.test_gpu_gated import run_gated

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule,L", [("plain", 1), ("plain", 63), ("plain", 64), ("plain", 65), ("plain", 200),
                                    ("gated", 64), ("gated", 200), ("fused", 64), ("fused", 200)])
@pytest.mark.parametrize("dtype,dk,dv,H", [("f32", 64, 64, 2), ("f32", 32, 64, 3), ("f32", 64, 32, 2), ("bf16", 64, 64, 2), ("bf16", 64, 128, 2),
                                           ("bf16", 128, 64, 2), ("bf16", 128, 128, 2), ("bf16", 256, 256, 1)])
def test_every_width_gives_the_same_bits(dtype, dk, dv, H, L, rule):
    inp = make_inputs(77 + L, B=1, L=L, H=H, dk=dk, dv=dv, dtype=dtype, with_initial_state=True, with_dfinal_state=True)
    label = "width %s %s %dx%d L=%d" % (rule, dtype, dk, dv, L)
    g = make_gate(3, inp.beta.shape)
    if rule == "plain":
        check_fwd_bwd(inp, label=label)
    elif rule == "gated":
        run_gated(inp, g, label=label)
    else:
        inp = make_pre_activations(3, inp)
        run_fused(inp, label)
    d = dev_inputs(inp)
    d["g"] = torch.from_numpy(g).cuda()
    f = lambda n: getattr(dn, "deltanet_" + {"plain": "", "gated": "gated_", "fused": "fused_"}[rule] + n)

    def passes(n):
        x = {k: v.expand(n, *v.shape[1:]).contiguous() for k, v in d.items() if v is not None}
        args = [x[k] for k in ("q", "k", "v", "beta") + (("g",) if rule == "gated" else ())]
        o, ST = f("fwd")(*args, x["S0"])
        grads = f("bwd")(*args, x["d_o"], x["S0"], x["dST"])
        o2, ST2, saved = f("fwd_save")(*args, x["S0"])
        grads2 = f("bwd_saved")(*args, x["d_o"], saved, x["dST"])
        torch.cuda.synchronize()
        return [o, ST, *grads, o2, ST2, *grads2]

    one = passes(1)
    chains = [256 * 32 // dv, 256 * 64 // dv]  # as many as fill the chip with 32, and with 64, columns per workgroup
    for n in chains:
        for i, (a, b) in enumerate(zip(one, passes(n // H))):
            assert torch.equal(a.expand_as(b), b), (n, i)


@pytest.mark.parametrize("rule", ["plain", "gated", "fused"])
@pytest.mark.parametrize("dtype,d,L", [("bf16", 128, 4096), ("bf16", 64, 4096), ("f32", 64, 512)])
def test_cut_sequence_equals_the_uncut_one(dtype, d, L, rule):
    """A long dense sequence of few heads is cut into segments; the same tokens as a packed batch of one sequence are not.  The two
    differ by the rounding of the segments' start states: each tensor within four times the error it has against 64 bits."""
    H = 2
    x = dev_inputs(make_inputs(8, B=1, L=L, H=H, dk=d, dv=d, dtype=dtype, with_initial_state=True, with_dfinal_state=True))
    args = [x[k] for k in ("q", "k", "v", "beta")]
    if rule == "gated":
        args.append(torch.log(0.9 + 0.1 * torch.rand(1, L, H, generator=torch.Generator().manual_seed(3))).cuda())
    f = lambda n: getattr(dn, "deltanet_" + {"plain": "", "gated": "gated_", "fused": "fused_"}[rule] + n)
    flat, cu = [a[0] for a in args], torch.tensor([0, L], dtype=torch.int32, device="cuda")
    o, ST, saved = f("fwd_save")(*args, x["S0"])
    cut = [o[0], ST, *[t[0] if t.dim() > 2 and t.shape[0] == 1 and t.shape[1] == L else t for t in f("bwd_saved")(*args, x["d_o"], saved, x["dST"])]]
    again = [t[0] if t.dim() > 2 and t.shape[0] == 1 and t.shape[1] == L else t for t in f("bwd")(*args, x["d_o"], x["S0"], x["dST"])]
    whole = [*f("fwd")(*flat, x["S0"], cu_seqlens=cu), *f("bwd")(*flat, x["d_o"][0], x["S0"], x["dST"], cu_seqlens=cu)]
    torch.cuda.synchronize()
    bound = 3e-2 if dtype == "bf16" and rule == "gated" else 2e-2 if dtype == "bf16" else 4e-6
    for i, (a, b) in enumerate(zip(cut, whole)):
        a, b = a.double().reshape(b.shape), b.double()
        assert (a - b).norm() <= bound * b.norm(), (i, float((a - b).norm() / b.norm()))
    for i, (a, b) in enumerate(zip(cut[2:], again)):
        assert torch.equal(a, b), i
