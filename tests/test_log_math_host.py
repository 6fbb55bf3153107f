"""Host checks of the log number system's exponentials and logarithms
(paper_1408_1664_amd/csrc/bn_math.h): errors in units of the last place against
long double, over the kernels' ranges (tests/native/math_check.cpp, built with
g++ here)."""
import os
import shutil
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_log_math():
    src = os.path.join(HERE, "native", "math_check.cpp")
    with tempfile.TemporaryDirectory() as td:
        exe = os.path.join(td, "math_check")
        subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-o", exe, src], check=True)
        r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "FAIL" not in r.stdout
    assert r.stdout.count("ok  ") == 24
