"""Host checks on the kernel sources: rules that a run of the kernels does not reliably show when they are broken."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2011_09208_amd", "csrc")


def asm_statements(text):
    """(template, outputs) of every inline-assembly statement."""
    for m in re.finditer(r"asm\s+volatile\s*\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = text[i]
            if c == '"' and text[i - 1] != "\\":
                quoted = not quoted
            depth += 0 if quoted else (c == "(") - (c == ")")
            i += 1
        body = text[m.end():i - 1]
        strings = re.match(r'\s*((?:"(?:[^"\\]|\\.)*"\s*)+)', body)
        rest = body[strings.end():]
        outputs = rest.split(":")[1].strip() if ":" in rest else ""
        yield strings.group(1), outputs


def test_asm_statements_are_found():
    got = list(asm_statements('asm volatile("a %0\\n" "b" : "=v"(x), "+v"(y) : "s"(f(z)) : "memory"); asm volatile("c" ::: "memory");'))
    assert [o for _, o in got] == ['"=v"(x), "+v"(y)', ""]


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip"))),
                         ids=os.path.basename)
def test_no_load_in_flight_has_an_output_register(path):
    """The compiler takes an output of inline assembly as written when the statement ends.  A load that is still in
    flight then may overwrite whatever the register holds by the time its data arrives."""
    for template, outputs in asm_statements(open(path).read()):
        if re.search(r"\b(buffer|global|flat|scratch|ds|s)_load|\bds_read", template) and outputs:
            assert "s_waitcnt" in template.rsplit("load", 1)[1], (os.path.basename(path), template)
