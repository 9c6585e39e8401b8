"""The bf16 chunk kernel whose tiles travel straight to the LDS, where a workgroup walks over several (chunk, head) tiles: the transfers of the next
one are under way while a tile is worked on, in the buffer that it is not in.  Tile counts around one and two per workgroup, an odd number, and
chunks of 1, 63 and 64 rows (rows past the end arrive as zeros)."""
import numpy as np
import pytest

from paper_2406_06484_amd.synth import make_gate, make_inputs, make_pre_activations
from tests.gpu_util import check_fwd_bwd, gpu_bwd
from tests.test_gpu_fused import run_fused
from tests.test_gpu_gated import run_gated

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule", ["plain", "gated", "fused"])
@pytest.mark.parametrize("dk,dv,B,L,H", [(128, 128, 1, 129, 86), (128, 128, 2, 127, 171), (128, 64, 1, 64, 257), (128, 64, 1, 129, 257), (64, 128, 1, 65, 140),
                                         (64, 64, 1, 64, 513), (64, 64, 3, 191, 115)])
def test_walks_of_several_tiles(dk, dv, B, L, H, rule):
    inp = make_inputs(40 + dk + 2 * dv + L, B=B, L=L, H=H, dk=dk, dv=dv, dtype="bf16", with_initial_state=True, with_dfinal_state=True)
    label = "%s %dx%d, %d tiles" % (rule, dk, dv, B * ((L + 63) // 64) * H)
    if rule == "plain":
        check_fwd_bwd(inp, label=label)
    elif rule == "gated":
        run_gated(inp, make_gate(5, inp.beta.shape, lo=0.8, hi=1.0), label=label)
    else:
        run_fused(make_pre_activations(6, inp), label)


def test_packed_walk_ends_before_the_grid_bound():
    """Short sequences: the walk's upper bound on the number of chunks is far above their number, and most chunks are ragged."""
    lens = np.array([1, 64, 65, 0, 130, 7, 63, 128, 33] * 6)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    check_fwd_bwd(make_inputs(91, H=9, dk=128, dv=128, dtype="bf16", with_initial_state=True, with_dfinal_state=True, cu_seqlens=cu), label="packed walk")


LENS = np.array([1, 64, 65, 0, 130, 7, 63, 128, 33] * 6)


def _mask(beta, first):
    """Zero, tiny and negative betas in two of three heads, [tokens, H]; `first`: the tokens that sequences begin with.  One head's tiles have a few rows of
    each kind (in the first chunk, across its end, in a ragged last one), the next one's first chunks have no other rows, the third one's have none."""
    tokens, H = beta.shape
    few, all_ = np.arange(H) % 3 == 1, np.arange(H) % 3 == 2
    for s in first:
        for lo, hi, value in ((3, 4, 0.0), (60, 70, 0.0), (80, 81, 2.0 ** -41), (81, 82, 2.0 ** -39), (128, 129, 0.0)):
            beta[s + lo:s + hi, few] = value
        beta[s + 90:s + 95, few] *= -1.0
        beta[s + 100:s + 101, few] = -2.0 ** -60
        beta[s:s + 64, all_] = 0.0


@pytest.mark.parametrize("rule", ["plain", "gated"])
@pytest.mark.parametrize("dk,dv,B,L,H", [(128, 128, 1, 129, 120), (128, 128, 3, 127, 120), (128, 64, 1, 129, 257), (64, 128, 2, 129, 100), (64, 64, 3, 191, 115)])
def test_walks_over_masked_and_unmasked_tiles(dk, dv, B, L, H, rule):
    """Masked rows edit a tile, store dv and wait at barriers of their own while the next tile travels."""
    inp = make_inputs(140 + dk + 2 * dv + L, B=B, L=L, H=H, dk=dk, dv=dv, dtype="bf16", with_initial_state=True, with_dfinal_state=True)
    for b in inp.beta:
        _mask(b, [0])
    label = "masked walk %s %dx%d, %d tiles" % (rule, dk, dv, B * ((L + 63) // 64) * H)
    if rule == "gated":
        run_gated(inp, make_gate(5, inp.beta.shape, lo=0.8, hi=1.0), label=label)
    else:
        check_fwd_bwd(inp, label=label)
        _, gk, gv, _, _ = gpu_bwd(inp)
        zero = inp.beta == 0
        assert zero.any() and not gk[zero].any() and not gv[zero].any()


@pytest.mark.parametrize("rule", ["plain", "gated", "fused"])
@pytest.mark.parametrize("dk,dv", [(128, 128), (128, 64), (64, 64)])
def test_packed_walks_with_masked_rows(dk, dv, rule):
    cu = np.concatenate([[0], np.cumsum(LENS)]).astype(np.int32)
    inp = make_inputs(191, H=9, dk=dk, dv=dv, dtype="bf16", with_initial_state=True, with_dfinal_state=True, cu_seqlens=cu)
    label = "masked packed walk %s %dx%d" % (rule, dk, dv)
    if rule == "fused":
        pre = make_pre_activations(7, inp)
        few = np.arange(9) % 3 == 1
        pre.beta[5::11, few], pre.beta[60:140, few] = -400.0, -120.0
        return run_fused(pre, label)
    _mask(inp.beta.reshape(-1, 9), [0, 1, 65, 130, 260, 1000, 2000])
    if rule == "gated":
        run_gated(inp, make_gate(6, inp.beta.shape, lo=0.8, hi=1.0), label=label)
    else:
        check_fwd_bwd(inp, label=label)
