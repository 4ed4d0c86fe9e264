"""How the update of moving bodies' masks is cut into launches, on the CPU."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1812_05401_amd", "csrc")


def test_the_nodes_of_a_launch_fit_an_int(tmp_path):
    exe = str(tmp_path / "place_plan_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, "-o", exe, os.path.join(HERE, "place_plan_check.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout
