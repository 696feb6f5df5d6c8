"""State that a handle builds on first use (the network's graph) is kept only when it is complete, on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_04263_amd", "csrc")


def test_a_failed_build_leaves_nothing(tmp_path):
    exe = str(tmp_path / "once_check")
    subprocess.run(["g++", "-O1", "-g", "-fsanitize=address,undefined", "-std=c++17", "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "once_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr


def test_the_graph_is_stored_by_it_alone():
    text = open(os.path.join(CSRC, "learned.hip")).read()
    assert text.count("build_once(h->learned,") == 1
    assert "h->learned =" not in text and "learned = L" not in text
