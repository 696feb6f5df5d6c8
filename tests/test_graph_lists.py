"""Host side of the network's graph kernels: their work lists and look-ahead indices where the entries of a
matrix end at the int32 limit, on the CPU (tests/native/pieces_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_04263_amd", "csrc")


def test_indices_at_the_end_of_the_range(tmp_path):
    exe = str(tmp_path / "pieces_check")
    subprocess.run(["g++", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=undefined", "-std=c++17",
                    "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "native", "pieces_check.cpp"), os.path.join(CSRC, "host_prep.cpp"),
                    os.path.join(CSRC, "host_parallel.cpp"), "-lpthread", "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
