"""The panel kernel's planning code (csrc/host_plan.h) under the host compiler's
sanitizers (tests/host/panel_plan_check.cpp).  No GPU is involved."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_panel_plan_under_asan_ubsan(tmp_path):
    exe = str(tmp_path / "panel_plan_check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wall",
           "-Wextra", "-Werror", os.path.join(HERE, "host", "panel_plan_check.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "all panel plan checks passed" in run.stdout
