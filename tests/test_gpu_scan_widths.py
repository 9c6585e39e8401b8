"""The scans give 16, 32 or 64 state columns to a workgroup, by the number of chains.  The columns are independent, so copies of one
sequence, few or many, have to give the bits of the sequence alone, at the lengths where a chunk step can go wrong (one token, one
chunk less one token, one chunk, one more); the sequence alone is checked against the oracle."""
import pytest
import torch

import paper_2406_06484_amd as dn
from paper_2406_06484_amd.synth import make_inputs
from tests.gpu_util import check_fwd_bwd, dev_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("dtype,dk,dv,H", [("f32", 64, 64, 2), ("f32", 32, 64, 3), ("f32", 64, 32, 2), ("bf16", 64, 64, 2), ("bf16", 64, 128, 2),
                                           ("bf16", 128, 64, 2), ("bf16", 128, 128, 2), ("bf16", 256, 256, 1)])
def test_every_width_gives_the_same_bits(dtype, dk, dv, H, L):
    kw = dict(B=1, L=L, H=H, dk=dk, dv=dv, dtype=dtype, with_initial_state=True, with_dfinal_state=True)
    check_fwd_bwd(make_inputs(77 + L, **kw), label="width %s %dx%d L=%d" % (dtype, dk, dv, L))
    d = dev_inputs(make_inputs(77 + L, **kw))

    def passes(n):
        x = {k: v.expand(n, *v.shape[1:]).contiguous() for k, v in d.items() if v is not None}
        args = [x[k] for k in ("q", "k", "v", "beta")]
        o, ST = dn.deltanet_fwd(*args, x["S0"])
        g = dn.deltanet_bwd(*args, x["d_o"], x["S0"], x["dST"])
        o2, ST2, saved = dn.deltanet_fwd_save(*args, x["S0"])
        g2 = dn.deltanet_bwd_saved(*args, x["d_o"], saved, x["dST"])
        torch.cuda.synchronize()
        return [o, ST, *g, o2, ST2, *g2]

    one = passes(1)
    chains = [256 * 32 // dv, 256 * 64 // dv]  # as many as fill the chip with 32, and with 64, columns per workgroup
    for n in chains:
        for i, (a, b) in enumerate(zip(one, passes(n // H))):
            assert torch.equal(a.expand_as(b), b), (n, i)
