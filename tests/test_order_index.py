"""CPU unit test of the arc indices of the weight-ordered loop (``csrc/gr_order.h``)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2212_08200_amd", "csrc")


def test_largest_graph_stays_in_int32(tmp_path):
    exe = tmp_path / "order_index_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC,
                    os.path.join(ROOT, "tests", "order_index_test.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


def test_every_step_is_within_the_run():
    # the loops' steps past a row's end (e += step, and entries of a queue)
    with open(os.path.join(CSRC, "gr_order.hip")) as f:
        text = f.read()
    run = int(re.search(r"kOrderRun = (\d+);", open(os.path.join(CSRC, "gr_order.h")).read()).group(1))
    consts = {k: int(v) for k, v in re.findall(r"constexpr int (k\w+) = (\d+);", text)}
    # (the host's loop over chunks ends before it steps past the last arc)
    steps = [eval(x, {}, consts) for x in re.findall(r"\be \+= ([\w* ]+)\)", text) if x != "kOrderChunk"]
    assert len(steps) >= 3 and 8 <= max(steps) <= run
    assert "order_indexes(m)" in open(os.path.join(CSRC, "gr_api.cpp")).read()
