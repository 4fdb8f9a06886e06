"""Inline assembly names the registers it writes beside its outputs: m0 and vcc are the compiler's too."""
import os
import re

import pytest

from paper_2105_01827_amd.build import CSRC

FILES = [f for f in sorted(os.listdir(CSRC)) if f.endswith((".hip", ".h"))]


def _statements(text):
    """the arguments of every asm statement, as written"""
    for m in re.finditer(r"\basm\b\s*(?:volatile\b\s*)?\(", text):
        depth, at, quoted = 1, m.end(), False
        while depth:
            c = text[at]
            if c == '"':
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            at += 1
        yield text[m.end():at - 1]


def _unnamed(statement):
    """registers that are an instruction's destination in the template and no clobber"""
    parts = re.split(r':(?=(?:[^"]*"[^"]*")*[^"]*$)', statement)        # at the colons outside of strings
    clobbers = re.findall(r'"(\w+)"', parts[3]) if len(parts) > 3 else []
    lines = "".join(re.findall(r'"([^"]*)"', parts[0])).replace("\\t", "").split("\\n")
    return {r for line in lines for r in ("m0", "vcc") if re.search(rf"^\s*\w+\s+(?:[^,]+,\s*)?{r}\b", line) and r not in clobbers}


def test_the_check_itself():
    assert _unnamed('"s_mov_b32 m0, %0\\n\\ts_nop 0" : : "s"(to), "n"(AT)') == {"m0"}
    assert _unnamed('"s_mov_b32 m0, %0" : : "s"(to) : "m0"') == set()
    assert _unnamed('"v_mad_i64_i32 %0, vcc, %1, 1, %0" : "+v"(H) : "v"(L)') == {"vcc"}
    assert _unnamed('"" : "+v"(tid)') == set()


@pytest.mark.parametrize("name", FILES)
def test_written_registers_are_named(name):
    found = list(_statements(open(os.path.join(CSRC, name)).read()))
    assert name != "gala_conv_mfma.hip" or found
    for statement in found:
        assert not _unnamed(statement), statement
