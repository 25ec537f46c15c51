"""The mixing launch's split rule on the CPU: tests/host/test_split.cpp with
lloid_plan.cpp under the address and undefined-behaviour sanitizers."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_16416_amd", "csrc")


def test_split_rule(tmp_path):
    exe = str(tmp_path / "test_split")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", CSRC, os.path.join(ROOT, "tests", "host", "test_split.cpp"),
                    os.path.join(CSRC, "lloid_plan.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
