"""The look-ahead's range test wraps without signed overflow (checked by the
compiler, in constant expressions)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_range_test_is_a_constant_expression():
    src = os.path.join(HERE, "host", "in_range_check.cpp")
    r = subprocess.run([HIPCC, "-std=c++17", "-fsyntax-only", src], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
