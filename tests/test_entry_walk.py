"""The kernels that walk CSR entries (csrc/entry_walk.hpp) on the largest
graphs the library takes, compiled with the host C++ compiler from the same
header and run on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_entries_stay_in_range(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path / "entry_walk_check"
    subprocess.run([cxx, "-std=c++17", "-O1", "-fwrapv", "-I", os.path.join(ROOT, "paper_2310_11222_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "entry_walk_check.cpp"), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "FAIL" not in r.stdout
