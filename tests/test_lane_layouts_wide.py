"""The lane layouts of the wide blocks (512 and 1024 threads), on the CPU: the
cells of a tile covered exactly once, one owner per staged cell, and in FP32
32 distinct LDS banks per half-wave."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_wide_blocks_cover_their_tiles(tmp_path):
    exe = tmp_path / "lane_layouts_wide_check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                           "-I", os.path.join(ROOT, "paper_1909_04153_amd", "csrc"),
                           os.path.join(ROOT, "tests", "lane_layouts_wide_check.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.count("cells") == 4 and r.stdout.count("staging") == 12, r.stdout
