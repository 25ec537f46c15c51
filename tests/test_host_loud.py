"""The bits of a conditioned block's loud samples on the CPU: ranges of every
length, also of many words, against a scan (tests/host/test_loud.cpp, under the
address and undefined-behaviour sanitizers)."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_16416_amd", "csrc")


def test_loud_ranges(tmp_path):
    exe = str(tmp_path / "test_loud")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", CSRC, os.path.join(ROOT, "tests", "host", "test_loud.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
