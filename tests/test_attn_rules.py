"""The size rules of the attention and of the copies, checked at compile time (they are host code)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.parametrize("source", ["attn_rules_check.cpp", "copy_rules_check.cpp"])
def test_rules_hold_on_both_sides_of_their_lines(source):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    r = subprocess.run([gxx, "-std=c++17", "-Wall", "-Werror", "-fsyntax-only", os.path.join(HERE, "native", source)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
