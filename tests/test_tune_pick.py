"""The autotuner keeps what it measured: its choice among timed launch shapes, as a host program."""
import os
import shutil
import subprocess

import pytest


def test_pick_variant(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = str(tmp_path / "tune_pick_check")
    cmd = ["g++", "-O1", "-std=c++17", "-I", os.path.join(root, "paper_2107_03679_amd", "csrc"),
           os.path.join(root, "tests", "tune_pick_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr
