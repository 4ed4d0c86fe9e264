"""The strips that a lattice is cut into, on the CPU: the library's own plan over random lattices."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1812_05401_amd", "csrc")


def test_plans_cover_the_lattice_within_their_table(tmp_path):
    exe = str(tmp_path / "strip_plan_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, "-o", exe, os.path.join(HERE, "strip_plan_check.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout
