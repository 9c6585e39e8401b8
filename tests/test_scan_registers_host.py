"""The bf16 scans of 64 columns keep everything in registers: a spilled value comes back through memory in every chunk step, behind the stores
before it.  Read from the compiler's resource report (no GPU needed); the gated kernels hold the most."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2406_06484_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("d", [128, 256])
def test_the_scans_do_not_spill(d, tmp_path):
    src = tmp_path / "scans.hip"
    args = "<dn::bf16, %d, %d, true, 4>(dn::SeqMap, int, dn::Ptrs);\n" % (d, d)
    src.write_text('#include "dn_kernels.hpp"\n' + "".join("template __global__ void dn::%s%s" % (k, args) for k in ("k_scan_fwd_save", "k_scan_bwd")))
    out = subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w",
                          "--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-I", CSRC, "-c", str(src), "-o", str(tmp_path / "scans.o")],
                         check=True, capture_output=True, text=True).stderr
    spills = re.findall(r"Function Name: (\S+k_scan\S+)|VGPRs Spill: (\d+)", out)
    names, counts = [n for n, _ in spills if n], [int(c) for _, c in spills if c]
    assert len(names) == 2 and not any(counts), counts
