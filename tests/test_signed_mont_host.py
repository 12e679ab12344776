"""The signed Montgomery arithmetic of the kernels, compiled for the host and checked against
__int128 (no GPU): exact products, their bounds, the quotient estimates and chains of butterflies."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("planted", [0, 1, 2, 3, 4])
def test_signed_mont(tmp_path, planted):
    """Planted: a bound too tight by 1.5 q, 2.25 q or 0.56 q, and a wrong power of two expected."""
    exe = tmp_path / "check"
    subprocess.check_call(["g++", "-std=c++17", "-O2", f"-DPLANT={planted}",
                           "-I", os.path.join(ROOT, "paper_2012_01968_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host", "signed_mont_check.cpp"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert (out.returncode == 0) == (planted == 0), out.stdout + out.stderr
    assert out.stdout.rstrip().endswith(" failures") and ("\n0 failures" in "\n" + out.stdout) == (planted == 0)
