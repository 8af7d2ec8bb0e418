"""The division by 6 of the smoother (a multiplication and two fused multiply-adds) on the host."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_div6_is_the_correctly_rounded_quotient(tmp_path):
    exe = tmp_path / "div6_check"
    src = os.path.join(ROOT, "tests", "native", "div6_check.cpp")
    inc = os.path.join(ROOT, "paper_1103_6031_amd", "csrc")
    r = subprocess.run(["g++", "-O2", "-mfma", "-std=c++17", "-I", inc, src, "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert "mismatches 0" in r.stdout and r.returncode == 0, r.stdout


def test_div_const_is_the_correctly_rounded_quotient(tmp_path):
    exe = tmp_path / "div_const_check"
    src = os.path.join(ROOT, "tests", "native", "div_const_check.cpp")
    inc = os.path.join(ROOT, "paper_1103_6031_amd", "csrc")
    r = subprocess.run(["g++", "-O2", "-mfma", "-std=c++17", "-I", inc, src, "-o", str(exe)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert "mismatches 0" in r.stdout and r.returncode == 0, r.stdout
