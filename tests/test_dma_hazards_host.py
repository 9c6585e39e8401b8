"""The bf16 chunk kernel's transfers to the LDS are written in inline asm, where the compiler does not keep the hardware's distances and does not know
what is written.  No run can show a distance that is too short while the old value of the register happens to be right, so this reads the compiled code
(no GPU needed): five wait states between a write of a scalar register on the vector unit and a buffer access that reads it, and nobody else's use of M0."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2406_06484_amd", "csrc")


def _scalars(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)", operand)
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def _instructions(asm):
    """(opcode, operands) in program order, without labels, directives and comments"""
    for line in asm.splitlines():
        s = line.split(";")[0].strip()
        if s and not s.startswith((".", "#")) and not s.endswith(":") and re.match(r"[a-z]\w+( |$)", s):
            op, _, rest = s.partition(" ")
            yield op, [w for part in rest.split(",") for w in part.split()]


def _read_too_early(asm):
    """Buffer accesses whose scalar operands were written on the vector unit fewer than five wait states before (an instruction is one, s_nop N is N + 1)"""
    bad, before = [], []
    for op, words in _instructions(asm):
        if op.startswith("buffer_"):
            reads, states = set().union(*map(_scalars, words)), 0
            for o, w in reversed(before):
                if states >= 5:
                    break
                if o.startswith("v_") and reads & _scalars(w[0]):
                    bad.append("%s %s, %d wait states, %s %s" % (o, " ".join(w), states, op, " ".join(words)))
                states += int(w[0], 0) + 1 if o == "s_nop" else 1
        before = before[-5:] + [(op, words)]
    return bad


def test_the_reader_sees_a_distance_that_is_too_short():
    near = "\tv_readlane_b32 s7, v1, 3\n\ts_mov_b32 m0, s2\n\ts_nop %d\n\tbuffer_load_dwordx4 v3, s[8:11], s7 offen nt lds ; note\n"
    assert _read_too_early(near % 0) and _read_too_early(near % 2) and not _read_too_early(near % 3)
    assert _read_too_early((near % 2).replace("s7, v1", "s9, v1")) and not _read_too_early((near % 2).replace("s7, v1", "s12, v1"))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("dk,dv", [(128, 128), (128, 64), (64, 128), (64, 64)])
def test_transfers_to_the_lds(dk, dv, tmp_path):
    src = tmp_path / "chunk.hip"
    src.write_text('#include "dn_launch.hpp"\n' + "".join(
        "template __global__ void dn::k_bwd_local<dn::bf16, %d, %d, dn::%s>(dn::SeqMap, int, dn::Ptrs, int);\n" % (dk, dv, v)
        for v in ("VAR_PLAIN", "VAR_GATED", "VAR_PROLOGUE")))
    asm = subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-w",
                          "--offload-device-only", "-S", "-I", CSRC, str(src), "-o", "-"], check=True, capture_output=True, text=True).stdout
    code = list(_instructions(asm))
    transfers = [i for i, (op, w) in enumerate(code) if op.startswith("buffer_load") and "lds" in w]
    assert len(transfers) >= 3 * 20
    assert not _read_too_early(asm)
    # M0 is written two instructions before each transfer, and nowhere else
    assert [i for i, (_, w) in enumerate(code) if "m0" in w] == [i - 2 for i in transfers]
