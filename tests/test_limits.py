"""The host code's decisions that need no device (sdp_limits.h), compiled with
the host compiler and run here."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_limits(tmp_path):
    exe = tmp_path / "limits_check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                           "-I", os.path.join(ROOT, "paper_2609_34162_amd", "csrc"),
                           os.path.join(ROOT, "tests", "c", "limits_check.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
