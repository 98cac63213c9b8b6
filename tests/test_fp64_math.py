"""The kernels' double-precision reciprocal, division, roots and face velocity
(the header they include, compiled for the host and started from
approximations as coarse as the hardware's): none is further from 113-bit
arithmetic than the correctly rounded operations in the definition's order."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_fp64_operations_round_no_worse_than_the_library_s(tmp_path):
    exe = tmp_path / "fp64_math_check"
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wall", "-Werror",
                           "-I", os.path.join(ROOT, "paper_1909_04153_amd", "csrc"),
                           os.path.join(ROOT, "tests", "fp64_math_check.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.endswith("\n0 failures\n"), r.stdout + r.stderr
