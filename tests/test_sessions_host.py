"""Host checks of the blocking calls' idle sessions (paper_1408_1664_amd/csrc/
bn_sessions.h) over a counting host device (tests/native/sessions_check.cpp,
built with g++ here): bounds, reuse, errors, memory that runs out, requests for
the memory, device resets, threads."""
import os
import shutil
import subprocess
import tempfile

import pytest

import paper_1408_1664_amd as bn

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_sessions():
    src = os.path.join(HERE, "native", "sessions_check.cpp")
    with tempfile.TemporaryDirectory() as td:
        exe = os.path.join(td, "sessions_check")
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread",
                        "-fsanitize=address,undefined", "-o", exe, src], check=True)
        r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "FAIL" not in r.stdout
    assert r.stdout.count("ok  ") == 19


def test_release_without_calls():
    bn.release_idle()
