"""The device memory pool's rules, on the CPU: pool.hip built with g++ against a fake
HIP of two devices (tests/fake_hip)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("pool") / "pool_check")
    csrc = os.path.join(ROOT, "paper_2608_05033_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-I", os.path.join(ROOT, "tests", "fake_hip"),
                           "-I", csrc, "-x", "c++", os.path.join(csrc, "pool.hip"),
                           os.path.join(ROOT, "tests", "pool_check.cpp"), "-o", exe])
    return exe


@pytest.mark.parametrize("case", ["devices_apart", "idle_first", "all_memory", "bounded", "threads"])
def test_pool(check, case):
    run = subprocess.run([check, case], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr
