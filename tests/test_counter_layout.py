"""The layout of event counters, on the CPU (tests/counter_layout.cpp against the library's own graph.cpp)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.join(HERE, "..")
CSRC = os.path.join(ROOT, "paper_2604_13327_amd", "csrc")


def test_counters_of_plans(tmp_path):
    exe = tmp_path / "counter_layout"
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-o", str(exe),
                           os.path.join(HERE, "counter_layout.cpp"), os.path.join(CSRC, "graph.cpp")])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout + out.stderr
