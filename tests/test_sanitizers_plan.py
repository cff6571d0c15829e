"""Address and undefined-behaviour sanitizer run of plan construction: the
host code of the library on a stand-in HIP runtime (tests/sanitize/plan_driver.cpp),
which lays out plans of every size class, order, precision and level offset.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"), reason="toolchain unavailable")
def test_plan_layout_under_asan_ubsan(tmp_path):
    exe = str(tmp_path / "plan_driver")
    cmd = ["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-g", "-O1", "-fno-omit-frame-pointer", "-w",
           "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-o", exe,
           os.path.join(ROOT, "paper_2606_13793_amd", "csrc", "fmm_api.cpp"),
           os.path.join(ROOT, "tests", "sanitize", "plan_driver.cpp")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600, env=env)
    out = r.stdout + r.stderr
    assert "runtime error" not in out and "AddressSanitizer" not in out and "LeakSanitizer" not in out, out
    assert r.returncode == 0 and "plans laid out" in out, out
