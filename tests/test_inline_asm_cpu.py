"""Instructions written as inline asm.  The compiler neither sees what such an
instruction is nor pads it: it may stand only where its result can be read by
the next instruction.  On gfx950 a dot product's (like a matrix product's or a
transcendental's) can not be, by another kind of instruction, for three wait
states, so those come from the compiler's builtins.  So do packed subtracts,
whose operands are uniform in one kernel and the lanes' own in another: an asm
operand is one or the other.
"""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2310_15668_amd", "csrc")

# 32-bit integer instructions without a wait of their own
PLAIN = {"v_and_or_b32", "v_sub_u32_e64", "v_mad_u32_u24"}
# times instructions; what they compute is not used
TIMING_ONLY = {"calibrate.hip"}


def _asm_instructions():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        if not path.endswith((".hip", ".h")) or os.path.basename(path) in TIMING_ONLY:
            continue
        with open(path) as f:
            text = f.read()
        for m in re.finditer(r"\basm\s*(?:volatile)?\s*\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", text):
            body = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1)))
            for line in re.split(r"\\n(?:\\t)?", body):
                if line.strip():
                    yield os.path.basename(path), line.split()[0]


def test_only_plain_instructions():
    found = list(_asm_instructions())
    assert found  # the pattern still matches the sources
    assert [x for x in found if x[1] not in PLAIN] == []
