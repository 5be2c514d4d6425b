"""The size rules of the attention, checked at compile time (they are host code)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_rules_hold_on_both_sides_of_their_lines():
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    r = subprocess.run([gxx, "-std=c++17", "-Wall", "-Werror", "-fsyntax-only", os.path.join(HERE, "native", "attn_rules_check.cpp")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
