"""The host runtime on the CPU (tests/host/test_runtime.cpp) with test doubles
of the HIP runtime and the kernel launches (tests/host/fake_hip.cpp), whose
streams run their work only when they are waited for: what a call reads and
writes, and when."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_16416_amd", "csrc")
HOST = os.path.join(ROOT, "tests", "host")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")), reason="no HIP headers")
def test_runtime_over_test_doubles(tmp_path):
    exe = str(tmp_path / "test_runtime")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(ROCM, "include"), "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), "-include", os.path.join(HOST, "fake_hip.h"),
                    os.path.join(HOST, "test_runtime.cpp"), os.path.join(HOST, "fake_hip.cpp"),
                    os.path.join(CSRC, "lloid_host.cpp"), os.path.join(CSRC, "lloid_plan.cpp"), "-lpthread", "-o", exe],
                   check=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:alloc_dealloc_mismatch=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
