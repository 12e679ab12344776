"""The launch rules of automatic plans, compiled with g++ from the header that the library uses (no
GPU): which launches take which split."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launch_rules(tmp_path):
    exe = tmp_path / "check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2012_01968_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host", "launch_rules_check.cpp"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.rstrip().endswith("0 failures")
