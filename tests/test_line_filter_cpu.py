"""The line filter's per-lane functions, compiled for the host from the
kernels' own headers (tests/cpu/hip gives the device names)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2305_01537_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    from paper_2305_01537_amd.build import HIPCC
    clang = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(HIPCC))), "lib", "llvm", "bin", "clang++")
    exe = str(tmp_path_factory.mktemp("cpu") / "line_filter_check")
    subprocess.run([clang, "-std=c++20", "-O1", "-mfma", "-ffp-contract=fast", "-pthread", "-Wno-everything", "-I", os.path.join(HERE, "cpu"), "-I", CSRC,
                    os.path.join(HERE, "cpu", "line_filter_check.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("name", ["sharp", "exponential", "radix3_lines", "other_lines"])
def test_line_filter(program, name):
    """sharp: a mode is kept exactly when |q| <= c, for cutoffs up to three
    units of the last place around every integer, at every line length, in
    both forms of the mask.  exponential: every factor is min(1, e^{c - |q|}) to
    the roundings that form it, in all three forms.  radix3_lines and
    other_lines: whole lines are no further from the exact filter on average
    than with every twiddle multiplied in by itself."""
    r = subprocess.run([program, name], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
