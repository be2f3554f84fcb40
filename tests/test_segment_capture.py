"""The no-allocation segment call's launches (syev3_noalloc.hip) against a
model of a stream and of graph capture, host code only, under
AddressSanitizer and UndefinedBehaviorSanitizer: eager and captured calls of
every size solve exactly their own requests.  No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_captured_and_eager_calls_solve_their_own_requests(tmp_path):
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip"):
        pytest.skip("g++ or the HIP headers not available")
    exe = str(tmp_path / "segment_capture")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer",
                           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1806_06698_amd", "csrc"),
                           "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           os.path.join(ROOT, "tests", "segment_capture_driver.cpp"),
                           "-o", exe])
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0",
               UBSAN_OPTIONS="print_stacktrace=1")
    p = subprocess.run([exe], capture_output=True, text=True, timeout=600, env=env)
    assert p.returncode == 0, p.stdout + p.stderr
    assert ", 0 failures" in p.stdout
