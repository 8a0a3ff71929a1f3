"""Which tile shape a merge runs (host replay)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_forced_tuned_and_default_shapes(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/bin/amdclang++"
    if not os.path.exists(cxx):
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "merge_shape")
    subprocess.run([cxx, "-O1", "-std=c++17", os.path.join(HERE, "merge_shape.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.startswith("OK"), res.stdout + res.stderr
