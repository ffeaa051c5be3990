"""Inline assembly that writes a register by name says so: the compiler is free to use m0 and the rest around a
statement that does not name it.  No GPU needed."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_23258_amd", "csrc")


def _asm_statements(text):
    for m in re.finditer(r"\basm\s+volatile\s*\(", text):
        depth, i = 1, m.end()
        in_string = False
        while depth:
            ch = text[i]
            if ch == '"' and text[i - 1] != "\\":
                in_string = not in_string
            elif not in_string:
                depth += (ch == "(") - (ch == ")")
            i += 1
        yield text[m.end(): i - 1]


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.h*"))), ids=os.path.basename)
def test_registers_written_by_name_are_clobbers(path):
    for body in _asm_statements(open(path).read()):
        code = body.split(":")[0]
        clobbers = body.rsplit(":", 1)[-1]
        # destinations of instructions that name a physical register (the first operand)
        for reg in re.findall(r"\b[sv]_\w+\s+(m0|vcc|exec|s\d+|v\d+)\s*,", code):
            assert f'"{reg}"' in clobbers, f"{os.path.basename(path)}: {body.strip()}"
