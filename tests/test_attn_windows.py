"""The windows of page ids an attention task goes through, on the CPU, for every page size a model may have (tests/attn_windows.cpp):
in 32 bits 4096 pages of 2^19 tokens are negative, and of 2^20 none."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2604_13327_amd", "csrc")


def test_windows_cover_every_chunk_for_every_page_size(tmp_path):
    exe = tmp_path / "attn_windows"
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC, "-o", str(exe), os.path.join(HERE, "attn_windows.cpp")])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout + out.stderr
