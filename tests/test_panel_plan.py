"""The panel kernel's planning code (csrc/host_plan.h) under the host compiler's
sanitizers (tests/host/panel_plan_check.cpp).  No GPU is involved."""

import os
import shutil
import subprocess

import pytest

from tests.panel_sizes import BATCHES, SINGLE

HERE = os.path.dirname(os.path.abspath(__file__))


pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("panel") / "panel_plan_check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wall",
           "-Wextra", "-Werror", os.path.join(HERE, "host", "panel_plan_check.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return exe


def test_panel_plan_under_asan_ubsan(exe):
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "all panel plan checks passed" in run.stdout


def _split(exe, sector, jobs):
    run = subprocess.run([exe, *map(str, sector), str(jobs)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stderr
    return [int(v) for v in run.stdout.split()]


def test_gpu_sizes_reach_every_variant(exe):
    """The sectors that the GPU tests run through the panel kernel still reach
    every variant, with as many rows per workgroup as it is built for."""
    for sector, want in SINGLE.items():
        got = _split(exe, sector, 0)
        assert tuple(got[:2]) == want and got[3] == 1, (sector, got)
        assert got[2] == (0 if sector == (14, 3, 3) else 1), (sector, got)
    for (sector, jobs), want in BATCHES.items():
        assert _split(exe, sector, jobs) == [*want, 1, 1], (sector, jobs)
    most = {}
    for variant, rows in [*SINGLE.values(), *BATCHES.values()]:
        most[variant] = max(rows, most.get(variant, 0))
    assert most == {0: 4, 1: 3, 2: 4, 3: 4, 4: 4, 5: 4, 6: 2}
