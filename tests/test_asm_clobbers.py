"""Inline assembly states what it writes: a register that an asm statement sets by name, without being
one of its outputs, is in its clobber list, or the compiler may keep a value of its own there.  And it keeps the waits
that the compiler does not see inside it: a vector-memory instruction must not read a scalar register within five wait
states of a vector instruction's write to it, which may stand right before the statement."""
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


def _parts(statement):
    """Its instructions, the constraints of its operands in order, its clobbers."""
    strings = re.findall(r'"((?:[^"\\]|\\.)*)"', statement)
    counts = [p.count('""') for p in re.sub(r'"(?:[^"\\]|\\.)*"', '""', statement).split(":")] + [0, 0, 0]
    code = " ".join(strings[:counts[0]]).replace("\\n", " \n ").replace("\\t", " ")
    clobbers = counts[0] + counts[1] + counts[2]
    return code, strings[counts[0]:clobbers], strings[clobbers:clobbers + counts[3]]


def _undeclared(statement):
    code, _, clobbers = _parts(statement)
    return sorted({r for r in WRITES.findall(code)} - set(clobbers))


def _unawaited(statement):
    """Operands that a vector-memory instruction takes from scalar registers which no scalar instruction of the statement
    has written before it."""
    code, constraints, _ = _parts(statement)
    written, found = set(), set()
    for line in code.split("\n"):
        if re.search(r"\b(global|buffer|flat|scratch)_", line):
            found |= {k for k in map(int, re.findall(r"%(\d+)", line)) if "s" in constraints[k]} - written
        written |= {int(k) for k in re.findall(r"\bs_[a-z0-9_]+\s+%(\d+)", line)}
    return sorted(found)


def test_the_scan_sees_an_undeclared_register():
    assert _undeclared(r'"s_mov_b32 m0, %1\n\tglobal_load %0" : : "v"(a), "s"(b) : "memory"') == ["m0"]
    assert _undeclared(r'"s_mov_b32 m0, %1\n\tglobal_load %0" : : "v"(a), "s"(b) : "m0", "memory"') == []


def test_the_scan_sees_an_unawaited_register():
    assert _unawaited(r'"s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load %0, %1" : : "v"(a), "s"(b), "s"(c) : "m0", "memory"') == [1]
    assert _unawaited(r'"s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load %1, %0" : "=&s"(t) : "v"(a), "s"(b), "s"(c) : "m0"') == []
    assert _unawaited(r'"s_mov_b32 m0, %1\n\tglobal_load %0, %1" : : "v"(a), "s"(b) : "m0", "memory"') == [1]
    assert _unawaited(r'"global_load %1, %0\n\ts_mov_b64 %0, %2" : "=&s"(t) : "v"(a), "s"(b)') == [0]


SOURCES = sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".inc", ".hpp")))


@pytest.mark.parametrize("name", SOURCES)
def test_loads_read_scalar_registers_that_scalar_instructions_wrote(name):
    with open(os.path.join(CSRC, name)) as f:
        for statement in _statements(f.read()):
            assert not _unawaited(statement), statement


@pytest.mark.parametrize("name", SOURCES)
def test_registers_written_by_name_are_clobbers(name):
    with open(os.path.join(CSRC, name)) as f:
        for statement in _statements(f.read()):
            assert not _undeclared(statement), statement
