"""The order of work in the launch that takes the layers whose hint missed: it ends, every unit in its turn, however few of its
workgroups the device holds at once (threads in the place of workgroups; see tickets_check.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_tickets_end_with_any_number_of_resident_workgroups(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "tickets_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-o", exe, os.path.join(HERE, "tickets_check.cpp")], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "tickets_check ok" in run.stdout, run.stdout + run.stderr
