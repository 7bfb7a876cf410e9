"""CPU unit test of the query server's queues for launches of their own
(``csrc/gr_sched.h``) with injected sizes."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launch_queues_share_the_budget(tmp_path):
    exe = tmp_path / "launch_queue_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2212_08200_amd", "csrc"),
                    os.path.join(ROOT, "tests", "launch_queue_test.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
