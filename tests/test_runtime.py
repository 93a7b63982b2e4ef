"""The host runtime (paper_2607_20125_amd/csrc/hc_runtime.cpp) alone, on the CPU:
tests/c/runtime_check.cpp compiles it against a HIP runtime in host memory
(tests/c/fake_hip.h) whose launches check the buffers they are given, and makes
allocations and copies fail."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_20125_amd", "csrc")
HIP = "/opt/rocm/include"


@pytest.fixture(scope="module")
def runtime_check(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir(HIP):
        pytest.skip("g++ or the HIP headers are not available")
    exe = tmp_path_factory.mktemp("runtime") / "runtime_check"
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", "-Werror",
           "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-D__HIP_PLATFORM_AMD__", "-isystem", HIP, "-I", CSRC, "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "c", "runtime_check.cpp"),
           os.path.join(CSRC, "hc_runtime.cpp"), "-o", str(exe)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return str(exe)


@pytest.mark.parametrize("check", ["errors_are_reported_once", "shared_buffers_after_failed_growth",
                                   "first_attention_on_another_stream", "small_windows", "host_memory"])
def test_runtime(runtime_check, check):
    run = subprocess.run([runtime_check, check], capture_output=True, text=True, timeout=120,
                         env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert run.returncode == 0, run.stdout + run.stderr
    assert f"{check}: ok" in run.stdout
