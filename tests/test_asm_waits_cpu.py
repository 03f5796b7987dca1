"""Inline assembly keeps the distances that the compiler keeps elsewhere."""
import glob
import os
import re

from paper_2206_14735_amd import gosurf as G

CSRC = os.path.join(os.path.dirname(os.path.abspath(G.__file__)), "csrc")
VALU_SGPR_TO_VMEM = 5   # wait states from a vector write of a scalar register to its use as an address


def _blocks():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        for m in re.finditer(r"\basm\b[^;(]*\((.*?)\);", open(path).read(), re.S):
            text, *operands = m.group(1).split("\n      : ")
            lines = [x for s in re.findall(r'"([^"]*)"', text) for x in re.split(r"\\n(?:\\t)?", s) if x.strip()]
            kinds = re.findall(r'"([=&+]*[a-z]+)"\s*\(', " ".join(operands))
            yield os.path.basename(path), lines, kinds


def test_memory_instructions_keep_their_distance_from_scalar_inputs():
    found = 0
    for name, lines, kinds in _blocks():
        waits = 0
        for ins in lines:
            scalars = [int(k) for k in re.findall(r"%(\d+)", ins) if kinds[int(k)] == "s"]
            if re.match(r"(global|flat|scratch|buffer)_", ins) and scalars:
                found += 1
                assert waits >= VALU_SGPR_TO_VMEM, (name, ins, waits)
            nop = re.match(r"s_nop (\d+)", ins)
            waits += 1 + (int(nop.group(1)) if nop else 0)
    assert found >= 1   # the record scatter's conditional adds
