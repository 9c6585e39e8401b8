"""Lanes of one wavefront that exchange data through the LDS without a barrier need a fence between the stores and the loads: the
hardware keeps the order, the compiler does not have to.  No run can show a missing one while the compiled order happens to be
right, so this looks at what the compiler is told: the IR of the inverse, before optimisation (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2406_06484_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_the_inverse_fences_its_exchange_between_lanes(tmp_path):
    src = tmp_path / "inverse.hip"
    src.write_text('#include "dn_device.hpp"\nextern "C" __global__ void k(float *g) {\n    __shared__ __align__(16) float x[64 * 68];\n'
                   "    dn::tri_inverse_64(x, 68);\n    g[threadIdx.x] = x[threadIdx.x];\n}\n")
    ir = subprocess.run(["hipcc", "--offload-arch=gfx950", "-std=c++17", "-O0", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                         "--offload-device-only", "-S", "-emit-llvm", "-I", CSRC, str(src), "-o", "-"],
                        check=True, capture_output=True, text=True).stdout
    body = re.search(r"define [^\n]*tri_inverse_64.*?\n}", ir, re.S).group(0)
    # the merges start at the first call of mma16_lds; the fence stands before it, after the diagonal blocks' stores
    before = body[:body.index("mma16_lds")]
    fence = before.rindex('fence syncscope("wavefront") acq_rel')
    assert "store float" in before[:fence] and "store float" not in re.sub(r"store float[^\n]*addrspace\(5\)[^\n]*", "", before[fence:])
