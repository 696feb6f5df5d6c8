"""Threads that raise a kernel's dynamic LDS limit at the same time, on the CPU (tests/native/limit_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_04263_amd", "csrc")


def test_the_limit_never_falls_below_what_a_thread_asked_for(tmp_path):
    exe = str(tmp_path / "limit_check")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "limit_check.cpp"), "-lpthread", "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stdout + out.stderr
