"""Inline asm beside matrix instructions, read from the assembly that the build's own flags give.

The compiler does not see an asm statement as the vector instruction it holds, so it leaves
out the wait states that the hardware asks for between a vector write and an MFMA that reads
the register as A or B, and between an MFMA and a vector write over its C or D registers.  No
register that an asm statement writes may therefore be one of an MFMA nearby.  Compiled for
the device only; nothing is run on a GPU."""
import os
import re
import subprocess

import pytest

from paper_2607_08779_amd import build

NEAR = 20        # instructions: above the longest wait, that of a 16-pass MFMA's result

REG = re.compile(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)")


def regs(operand):
    found = set()
    for lo, hi, one in REG.findall(operand):
        found |= set(range(int(lo), int(hi) + 1)) if lo else {int(one)}
    return found


def instructions(path):
    """(kernel, opcode, operands, in an asm statement) of every instruction."""
    kernel, inside = "", False
    for line in open(path):
        s = line.split(";")[0].strip() if ";;#ASM" not in line else line.strip()
        if s.startswith(";;#ASMSTART"):
            inside = True
        elif s.startswith(";;#ASMEND"):
            inside = False
        elif s.endswith(":") and not s.startswith("."):
            kernel = s[:-1]
        elif s and not s.startswith((".", ";")) and not s.endswith(":"):
            op, _, rest = s.partition(" ")
            yield kernel, op, [p.strip() for p in re.split(r",(?![^\[]*\])", rest)], inside


def conflicts(path):
    """MFMAs that read, as A or B, what an asm statement wrote shortly before, or whose C or D
    an asm statement overwrites shortly after."""
    bad, recent, mfma, last = [], {}, [], None
    for i, (kernel, op, args, inside) in enumerate(instructions(path)):
        if kernel != last:
            recent, mfma, last = {}, [], kernel
        if op.startswith("v_mfma"):
            for r in regs(args[1]) | regs(args[2]):
                if i - recent.get(r, -NEAR) < NEAR:
                    bad.append((kernel, op, r))
            mfma = [m for m in mfma if i - m[0] < NEAR] + [(i, regs(args[0]) | regs(args[3]))]
        if inside and op.startswith("v_"):
            for r in regs(args[0]):
                recent[r] = i
                if any(i - at < NEAR and r in cd for at, cd in mfma):
                    bad.append((kernel, op, r))
        elif args and args[0] and not op.startswith(("s_", "buffer_store", "global_store", "ds_write")):
            for r in regs(args[0]):
                recent.pop(r, None)
    return bad


WITH_BOTH = ["gemm.hip", "skinny.hip"]      # and_or() (or dequant_part(), made of it) beside MFMA


def test_the_files_with_both_are_listed():
    found = []
    for src in build.sources():
        text = open(src).read()
        text += "".join(open(os.path.join(build.CSRC, h)).read() for h in re.findall(r'#include "((?:stream|tile)_\w+\.h)"', text))
        text = re.sub(r"//.*", "", text)
        if "_mfma_" in text and re.search(r"\b(and_or|dequant_part<.*>)\(", text):
            found.append(os.path.basename(src))
    assert found == WITH_BOTH


def test_the_scan_sees_both_hazards(tmp_path):
    asm = ("k:\n\t;;#ASMSTART\n\tv_and_or_b32 v7, v1, s0, v2\n\t;;#ASMEND\n\ts_nop 0\n"
           "\tv_mfma_f32_16x16x32_bf16 v[8:11], v[12:15], v[4:7], v[8:11]\n"
           "\t;;#ASMSTART\n\tv_and_or_b32 v9, v1, s0, v2\n\t;;#ASMEND\n")
    (tmp_path / "x.s").write_text(asm)
    assert [r for _, _, r in conflicts(tmp_path / "x.s")] == [7, 9]
    (tmp_path / "y.s").write_text(asm.replace("s_nop 0", "v_mov_b32_e32 v7, v7").replace("v9,", "v20,"))
    assert conflicts(tmp_path / "y.s") == []


@pytest.mark.parametrize("name", WITH_BOTH)
def test_no_mfma_meets_a_register_written_in_asm(name, tmp_path):
    out = str(tmp_path / "device.s")
    subprocess.run([build.hipcc(), *build.FLAGS, *build.FILE_FLAGS.get(name, build.VGPR_FORM), "--cuda-device-only",
                    "-S", os.path.join(build.CSRC, name), "-o", out], check=True, capture_output=True, timeout=600)
    assert "v_mfma" in open(out).read()
    bad = conflicts(out)
    assert not bad, f"{name}: {len(bad)} places, first {bad[0]}"
