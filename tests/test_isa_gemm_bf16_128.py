"""Static check of the compiled fragment reads of gemm_bf16_128.hip (CPU only:
hipcc cross-compiles it to gfx950 assembly).

The kernels read their fragments out of LDS in inline assembly, which the
compiler takes as done at once: it inserts no wait, and would be free to copy or
reuse a destination register while the read is in flight. The source keeps the
registers untouched up to a wait of its own. Checked in every kernel: between a
read and the next s_waitcnt lgkmcnt(0) no other instruction names its destination,
and no read is in flight across a label or a branch.
"""

import os
import re
import subprocess

import pytest

from paper_1603_04467_amd import build as B

pytestmark = pytest.mark.timeout(600)

SRC = "gemm_bf16_128.hip"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    path = os.path.join(tmp_path_factory.mktemp("isa"), SRC + ".s")
    cmd = [B._hipcc(), *B.FLAGS, *B.SOURCE_FLAGS.get(SRC, []), "--cuda-device-only", "-S", os.path.join(B.CSRC, SRC),
           "-o", path]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = open(path).read()
    return {m.group(1): text[m.end():text.index(".Lfunc_end", m.end())].splitlines()
            for m in re.finditer(r"^(_Z\S*gemm_bf16_128\S*):", text, re.M)}


def _vgprs(operands):
    regs = set()
    for m in re.finditer(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)", operands):
        regs |= set(range(int(m.group(1)), int(m.group(2)) + 1)) if m.group(1) else {int(m.group(3))}
    return regs


def _early_uses(lines):
    """(number of inline reads, the lines that touch one in flight)."""
    in_asm, flying, reads, bad = False, set(), 0, []
    for line in lines:
        if "#ASMSTART" in line or "#ASMEND" in line:
            in_asm = "#ASMSTART" in line
            continue
        s = line.split(";")[0].strip()
        if not s or (s.startswith(".") and not s.endswith(":")):
            continue
        if re.match(r"s_waitcnt\b.*lgkmcnt\(0\)", s):
            flying = set()
            continue
        if flying and (s.endswith(":") or s.startswith(("s_cbranch", "s_branch", "s_endpgm"))):
            bad.append(s)
            continue
        op, _, operands = s.partition(" ")
        if flying & _vgprs(operands):
            bad.append(s)
        if in_asm and op.startswith("ds_read"):
            reads += 1
            flying |= _vgprs(operands.split(",")[0])
    return reads, bad


def test_no_fragment_is_touched_in_flight(kernels):
    assert len(kernels) == 54  # 3 layouts x 6 outputs and epilogues x 3 tile and stage forms
    for name, lines in kernels.items():
        reads, bad = _early_uses(lines)
        # 24 reads of b128 fragments (two halves each where they are transposed): the first step's 8 and the loop's 16
        assert reads in (24, 36, 48), (name, reads)
        assert not bad, (name, bad[:4])


def test_the_check_sees_an_early_use():
    read = ["\t;;#ASMSTART", "\tds_read_b128 v[4:7], v1", "\t;;#ASMEND"]
    wait = ["\t;;#ASMSTART", "\ts_waitcnt lgkmcnt(0)", "\t;;#ASMEND"]
    assert _early_uses(read + ["\tv_mov_b32_e32 v2, v3"] + wait + ["\tv_mov_b32_e32 v2, v5"]) == (1, [])
    assert _early_uses(read + ["\tv_mov_b32_e32 v2, v5"] + wait)[1]
    assert _early_uses(read + ["\tv_add_u32_e32 v7, v2, v3"] + wait)[1]
    assert _early_uses(read + [".LBB0_2:"] + wait)[1]
