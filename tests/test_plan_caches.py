"""The rules for the caches and the sizes of big tiles, on the CPU under AddressSanitizer and
UBSan."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1910_00643_amd", "csrc")


def test_rules(tmp_path):
    exe = str(tmp_path / "plan_caches")
    cmd = ["g++", "-O1", "-g", "-std=c++17", "-Wall", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", "-static-libasan", "-I", CSRC, "-o", exe,
           os.path.join(ROOT, "tests", "plan_caches_driver.cpp"), os.path.join(CSRC, "slowmo_plan.cpp")]
    build = subprocess.run(cmd, capture_output=True, text=True)
    if build.returncode != 0 and "asan" in (build.stderr + build.stdout).lower():
        pytest.skip("this toolchain has no static AddressSanitizer runtime")
    assert build.returncode == 0, build.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
