"""Inline assembly states what it writes: a register that an asm statement sets by name, without being
one of its outputs, is in its clobber list, or the compiler may keep a value of its own there."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_22881_amd", "csrc")
# the destination of an instruction is its first operand
WRITES = re.compile(r"\b[sv]_[a-z0-9_]+\s+(m0|vcc|exec|scc|[sv]\d+|[sv]\[\d+:\d+\])\b")


def _statements(text):
    for m in re.finditer(r"\basm\s+volatile\s*\(", text):
        depth, i = 1, m.end()
        quoted = False
        while depth:
            c = text[i]
            if c == '"':
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            i += 1
        yield text[m.end():i - 1]


def _undeclared(statement):
    strings = re.findall(r'"((?:[^"\\]|\\.)*)"', statement)
    colons = re.sub(r'"(?:[^"\\]|\\.)*"', '""', statement).split(":")
    code = " ".join(strings[:colons[0].count('""')]).replace("\\n", " \n ").replace("\\t", " ")
    clobbers = strings[len(strings) - colons[3].count('""'):] if len(colons) > 3 else []
    return sorted({r for r in WRITES.findall(code)} - set(clobbers))


def test_the_scan_sees_an_undeclared_register():
    assert _undeclared(r'"s_mov_b32 m0, %1\n\tglobal_load %0" : : "v"(a), "s"(b) : "memory"') == ["m0"]
    assert _undeclared(r'"s_mov_b32 m0, %1\n\tglobal_load %0" : : "v"(a), "s"(b) : "m0", "memory"') == []


@pytest.mark.parametrize("name", sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".inc", ".hpp"))))
def test_registers_written_by_name_are_clobbers(name):
    with open(os.path.join(CSRC, name)) as f:
        for statement in _statements(f.read()):
            assert not _undeclared(statement), statement
