"""The chunk-local backward kernel at the rows where dbeta cannot be the quotient dV . Ut / beta^2: beta zero (masked tokens),
tiny or negative, alone, in runs across a chunk boundary, in a ragged last chunk, for every compiled head size and rule."""
import numpy as np
import pytest

from paper_2406_06484_amd.synth import make_gate, make_inputs
from tests.gpu_util import check_fwd_bwd
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
