"""The preparation of a brick under the thread order that a missing barrier would not survive, on the CPU.

Every thread of a brick's block decides from the brick's flag whether to clear its cells, and thread 0
replaces the flag.  The driver compiles the function's own text for the host and lets thread 0 run ahead of
all others as far as its barriers allow: the cells cleared and the flag left must be those of the modes."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def function_text(source, name):
    start = re.search(r"^__device__ __forceinline__ void " + name + r"\(", source, re.M).start()
    at = source.index("{", start)
    depth, end = 1, at + 1
    while depth:
        depth += {"{": 1, "}": -1}.get(source[end], 0)
        end += 1
    return source[start:end]


def test_every_thread_reads_the_flag_before_it_is_replaced(tmp_path):
    with open(os.path.join(ROOT, "paper_1504_02591_amd", "csrc", "recon_kernels.hpp")) as f:
        text = function_text(f.read(), "brick_prepare")
    src = tmp_path / "brick_prepare.inc"
    src.write_text(text + "\n")
    exe = tmp_path / "driver"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", f'-DBRICK_PREPARE_SOURCE="{src}"', "-o", str(exe),
                    os.path.join(ROOT, "tests", "brick_prepare_driver.cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
