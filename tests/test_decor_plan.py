"""Loads of the correlation reduction's substitution, checked on the CPU for every
number of rows (tests/cpp/decor_plan_check.cpp, built with g++)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_substitution_reads_rows_of_the_factor(tmp_path):
    exe = str(tmp_path / "decor_plan_check")
    src = os.path.join(HERE, "cpp", "decor_plan_check.cpp")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-o", exe, src], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "ALL OK" in r.stdout, r.stdout
