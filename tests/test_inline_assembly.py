"""Registers that inline assembly in the kernels names by itself are among its clobbers: the compiler may otherwise
keep a value of its own in them across the statement (m0: indexed register moves, messages, its own LDS loads)."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_04610_amd", "csrc")
REGISTER = re.compile(r"\b(m0|vcc|exec|scc)\b|\b([sv]\d+)\b|\b[sv]\[\d+:\d+\]")


def statements(text):
    """(template, the rest) of every asm statement: up to the closing parenthesis, strings skipped"""
    for m in re.finditer(r"\basm\s+volatile\s*\(|\basm\s*\(|__asm__\s*(?:volatile\s*)?\(", text):
        i, depth, quoted = m.end(), 1, False
        while depth:
            c = text[i]
            if c == '"' and text[i - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += {"(": 1, ")": -1}.get(c, 0)
            i += 1
        body = text[m.end():i - 1]
        t = re.match(r'\s*((?:"(?:[^"\\]|\\.)*"\s*)+)', body)
        yield t.group(1), body[t.end():]


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*"))), ids=os.path.basename)
def test_named_registers_are_clobbered(path):
    with open(path) as f:
        text = re.sub(r"//[^\n]*", "", f.read())
    for template, rest in statements(text):
        named = {m.group(0) for m in REGISTER.finditer(template.replace("\\n", " ").replace("\\t", " "))}
        missing = [r for r in named if f'"{r}"' not in rest]
        assert not missing, (template, missing)
