"""The load cursor of the register-held mixing kernel on the CPU: every ring
depth, windows of one to five tiles, runs that begin anywhere in a window
(tests/host/test_cursor.cpp, under the address and undefined-behaviour
sanitizers).  A tile at or past the run's end has no operand rows to read."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_16416_amd", "csrc")


def test_loads_end_with_the_run(tmp_path):
    exe = str(tmp_path / "test_cursor")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", CSRC, os.path.join(ROOT, "tests", "host", "test_cursor.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
