"""The scans with the most columns per workgroup keep everything in registers: a spilled value comes back through memory in every chunk step, behind the stores
before it.  Read from the compiler's resource report (no GPU needed); the gated kernels hold the most."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2406_06484_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("dtype,d,waves,gated", [("bf16", 128, 4, True), ("bf16", 256, 4, True), ("float", 64, 2, True), ("float", 64, 2, False)])
def test_the_scans_do_not_spill(dtype, d, waves, gated, tmp_path):
    src = tmp_path / "scans.hip"
    args = "<%s, %d, %d, %s, %d>(dn::SeqMap, int, dn::Ptrs" % (dtype if dtype == "float" else "dn::" + dtype, d, d, str(gated).lower(), waves)
    kernels = dict(k_scan_fwd_save=");\n", k_scan_bwd=");\n", k_scan_pair=", int);\n")
    if d <= 128:  # the passes over segments
        kernels.update(k_scan_state=", int);\n", k_scan_bwd_state=");\n")
    src.write_text('#include "dn_kernels.hpp"\n' + "".join("template __global__ void dn::%s%s%s" % (k, args, end) for k, end in kernels.items()))
    out = subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w",
                          "--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-I", CSRC, "-c", str(src), "-o", str(tmp_path / "scans.o")],
                         check=True, capture_output=True, text=True).stderr
    spills = re.findall(r"Function Name: (\S+k_scan\S+)|VGPRs Spill: (\d+)", out)
    names, counts = [n for n, _ in spills if n], [int(c) for _, c in spills if c]
    assert len(names) == len(kernels) and not any(counts), counts
