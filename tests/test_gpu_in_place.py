"""Gradient buffers that are also inputs (dq over q, dk over k, dv over v, dv over d_o): the same bits as with buffers of their own,
for every rule, kept and recomputed, with masked tokens, uncut and segmented scans, dense and packed."""
import numpy as np
import pytest
import torch

import paper_2406_06484_amd as dn
from paper_2406_06484_amd.synth import make_gate, make_inputs
from tests.gpu_util import dev_inputs

pytestmark = pytest.mark.gpu

CU = np.array([0, 0, 5, 69, 199, 262, 263, 263, 520], dtype=np.int32)


@pytest.mark.parametrize("over", ["q k v", "d_o", "k q", "dk over d_o"])
@pytest.mark.parametrize("kept", [True, False])
@pytest.mark.parametrize("rule", ["plain", "gated", "fused"])
@pytest.mark.parametrize("dtype,d,shape", [("f32", 64, dict(B=2, L=200)), ("bf16", 64, dict(B=2, L=200)), ("bf16", 128, dict(cu_seqlens=CU)),
                                           ("bf16", 128, dict(B=1, L=512)), ("bf16", 256, dict(B=2, L=130))])
def test_gradients_over_inputs(dtype, d, shape, rule, kept, over):
    inp = make_inputs(61, H=2, dk=d, dv=d, dtype=dtype, with_initial_state=True, with_dfinal_state=True, **shape)
    inp.beta.reshape(-1, 2)[::7] = 0.0
    t = dev_inputs(inp)
    extra = [torch.from_numpy(make_gate(3, inp.beta.shape)).cuda()] if rule == "gated" else []
    pre = {"plain": "", "gated": "gated_", "fused": "fused_"}[rule]
    f = lambda n: getattr(dn, "deltanet_%s%s" % (pre, n))

    def grads(alias):
        q, k, v, d_o = (t[n].clone() for n in ("q", "k", "v", "d_o"))
        kw = {}
        if alias == "q k v":
            kw = dict(dq=q, dk=k, dv=v)
        elif alias == "d_o":
            kw = dict(dv=d_o)
        elif alias == "k q":
            kw = dict(dq=k, dk=q)
        elif alias == "dk over d_o":
            kw = dict(dk=d_o, dv=k)
        args = [q, k, v, t["beta"]] + extra
        ckw = dict(cu_seqlens=t["cu"])
        if kept:
            _, _, saved = f("fwd_save")(*args, t["S0"], **ckw)
            return f("bwd_saved")(*args, d_o, saved, t["dST"], **kw, **ckw)
        return f("bwd")(*args, d_o, t["S0"], t["dST"], **kw, **ckw)

    want, got = grads(None), grads(over)
    torch.cuda.synchronize()
    for n, a, b in zip(("dq", "dk", "dv", "dbeta"), want, got):
        assert torch.equal(a, b), n
