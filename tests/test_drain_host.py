"""Calls that end by an error or an exception leave no stream at work on their
host buffers, and no pinned block that a stream may still write in the pool."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_streams_are_drained(tmp_path):
    exe = str(tmp_path / "drain_check")
    cmd = ["g++", "-O1", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "tests", "cpp", "hip_stub"),
           "-I", os.path.join(ROOT, "paper_1805_00475_amd", "csrc"),
           os.path.join(ROOT, "tests", "cpp", "drain_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
