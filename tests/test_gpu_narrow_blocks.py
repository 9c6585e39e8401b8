"""The scans of few chains own 16 or 32 state columns per workgroup instead of 64 (of 32 in fp32).  A batch of copies of one sequence, large enough for
the ordinary blocks, has to give the bits of the sequence alone: the tiles are formed by the same products in the same order."""
import numpy as np
import pytest
import torch

import paper_2406_06484_amd as dn
from paper_2406_06484_amd.synth import make_gate, make_inputs
from tests.gpu_util import check_fwd_bwd, dev_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule", ["plain", "gated", "fused"])
@pytest.mark.parametrize("dk,dv,H,L", [(64, 64, 3, 1), (64, 64, 8, 200), (64, 128, 5, 130), (128, 64, 9, 65), (128, 128, 3, 64), (128, 128, 16, 333)])
def test_narrow_equals_wide(dk, dv, H, L, rule):
    copies = 300 // H  # more than 256 workgroups with either block
    inp = make_inputs(40 + dk + dv + L, B=1, L=L, H=H, dk=dk, dv=dv, dtype="bf16", with_initial_state=True, with_dfinal_state=True)
    d = dev_inputs(inp)
    one = [d[n] for n in ("q", "k", "v", "beta")]
    if rule == "gated":
        one.append(torch.from_numpy(make_gate(4, inp.beta.shape, lo=0.8, hi=1.0)).float().cuda())
    d_o = torch.randn(1, L, H, dv, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16).cuda()
    dST = torch.randn(1, H, dk, dv, generator=torch.Generator().manual_seed(2)).cuda()
    pre = {"plain": "deltanet_", "gated": "deltanet_gated_", "fused": "deltanet_fused_"}[rule]
    f = lambda n: getattr(dn, pre + n)
    many = lambda x: x.expand(copies, *x.shape[1:]).contiguous()

    def passes(args, S0, do, dS):
        o, ST = f("fwd")(*args, S0)
        g = f("bwd")(*args, do, S0, dS)
        o2, ST2, saved = f("fwd_save")(*args, S0)
        g2 = f("bwd_saved")(*args, do, saved, dS)
        torch.cuda.synchronize()
        return [o, ST, *g, o2, ST2, *g2]

    few = passes(one, d["S0"], d_o, dST)
    lot = passes([many(x) for x in one], many(d["S0"]), many(d_o), many(dST))
    for i, (a, b) in enumerate(zip(few, lot)):
        assert torch.equal(many(a), b), i


def test_narrow_packed():
    cu = np.array([0, 0, 5, 69, 199, 262, 263, 263, 520], dtype=np.int32)
    for dk, dv in ((64, 128), (128, 128)):
        check_fwd_bwd(make_inputs(9, H=3, dk=dk, dv=dv, dtype="bf16", cu_seqlens=cu, with_initial_state=True, with_dfinal_state=True), label="narrow packed %dx%d" % (dk, dv))
