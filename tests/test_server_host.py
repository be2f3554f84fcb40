"""The server's host-staged requests (syev3_server.cpp) against a model of the
HIP runtime, host code only, under AddressSanitizer and
UndefinedBehaviorSanitizer: which buffers the kernel takes in place, how many
workgroups it may use, and that the runtime is not queried under the server's
lock.  No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_host_staged_requests(tmp_path):
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip"):
        pytest.skip("g++ or the HIP headers not available")
    exe = str(tmp_path / "server_host")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-pthread",
                           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1806_06698_amd", "csrc"),
                           "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           os.path.join(ROOT, "tests", "server_host_driver.cpp"), "-o", exe])
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0",
               UBSAN_OPTIONS="print_stacktrace=1")
    p = subprocess.run([exe], capture_output=True, text=True, timeout=600, env=env)
    assert p.returncode == 0, p.stdout + p.stderr
    assert "0 failures" in p.stdout
