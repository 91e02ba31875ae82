"""Rules of the device sources that no run of a kernel shows reliably."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2105_04006_amd", "csrc")


def asm_statements(text):
    """(template, output operands) of every asm statement, comments removed."""
    text = re.sub(r"//[^\n]*|/\*.*?\*/", "", text, flags=re.S)
    for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(", text):
        depth, quoted, end = 1, False, m.end()
        while depth:
            c = text[end]
            if c == '"' and text[end - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            end += 1
        body = text[m.end():end - 1]
        template = re.match(r'\s*((?:"(?:[^"\\]|\\.)*"\s*)+)', body)
        rest = body[template.end():]
        outputs = rest.split(":")[1] if ":" in rest else ""
        yield "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', template.group(1))), outputs.strip()


@pytest.mark.parametrize("name", sorted(os.listdir(CSRC)))
def test_no_instruction_of_inline_assembly_writes_a_register(name):
    """The compiler's hazard pass does not know what an instruction inside an asm
    statement writes: a matrix instruction that reads it may follow without the
    two wait states that it needs, and get the old value."""
    with open(os.path.join(CSRC, name)) as f:
        found = [(t, o) for t, o in asm_statements(f.read()) if t.strip() and o]
    assert not found, f"{name}: {found}"
