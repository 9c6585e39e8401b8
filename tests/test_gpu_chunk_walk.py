"""The bf16 chunk kernel whose tiles travel straight to the LDS, where a workgroup walks over several (chunk, head) tiles: the transfers of the next
one are under way while a tile is worked on, in the buffer that it is not in.  Tile counts around one and two per workgroup, an odd number, and
chunks of 1, 63 and 64 rows (rows past the end arrive as zeros)."""
import numpy as np
import pytest

from paper_2406_06484_amd.synth import make_gate, make_inputs, make_pre_activations
from tests.gpu_util import check_fwd_bwd
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
