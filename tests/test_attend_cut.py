"""How attention over a card is cut into tasks, over random shapes and class counts on the CPU, by the code that the device runs: where a wave takes one task
there are no more tasks than waves, a task is a whole number of load groups and fits its LDS, every row of every class belongs to one
task, and the partials fit the workspace."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_every_row_has_a_task_and_every_task_a_wave(tmp_path):
    exe = str(tmp_path / "attend_cut_drive")
    build = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wno-unknown-pragmas", "-o", exe, os.path.join(ROOT, "tests", "attend_cut_drive.cpp")], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-4000:]
    for seed in (1, 2):
        run = subprocess.run([exe, "40000", str(seed)], capture_output=True, text=True, timeout=300)
        assert run.returncode == 0, (run.stdout[-2000:], run.stderr[-2000:])
        assert "cut ok" in run.stdout
