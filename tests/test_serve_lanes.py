"""Forks, joins and the error path of a serving tick's lanes on the CPU, with
fake streams and a failure at each of a tick's calls in turn
(tests/cpp/serve_lanes_check.cpp, built with g++)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_lanes_and_error_path(tmp_path):
    exe = str(tmp_path / "serve_lanes_check")
    src = os.path.join(HERE, "cpp", "serve_lanes_check.cpp")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-o", exe, src], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "ALL OK" in r.stdout, r.stdout
