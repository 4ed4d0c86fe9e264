"""Host work spread over threads, on the CPU: done whole where a thread cannot be started."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1812_05401_amd", "csrc")


def test_work_is_done_where_a_thread_finds_no_memory(tmp_path):
    exe = str(tmp_path / "side_by_side_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", CSRC, "-o", exe, os.path.join(HERE, "side_by_side_check.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout + res.stderr
