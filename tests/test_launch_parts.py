"""The split of launches that would be more threads than HIP takes (no GPU needed)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_parts_cover_every_workgroup_once(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not installed")
    exe = str(tmp_path / "launch_parts")
    build = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror",
                            "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2508_01073_amd", "csrc"),
                            os.path.join(ROOT, "tests", "host", "launch_parts.cpp"), "-o", exe],
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert build.returncode == 0, build.stdout
    run = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert run.returncode == 0 and "launch parts: ok" in run.stdout, run.stdout
