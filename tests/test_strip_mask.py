"""Which mask entries the strip sweep reads, on the CPU: its rows and columns from the library's own functions."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1812_05401_amd", "csrc")


def test_every_mask_entry_lies_in_the_lattice(tmp_path):
    exe = str(tmp_path / "strip_mask_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, "-o", exe, os.path.join(HERE, "strip_mask_check.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout
