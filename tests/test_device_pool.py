"""The device memory pool's decisions on the host, with a stand-in device
(device_pool_check.cpp)."""

import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2604_18886_amd", "csrc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("pool") / "device_pool_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", CSRC,
                           os.path.join(HERE, "device_pool_check.cpp"), "-o", exe])
    return exe


@pytest.mark.parametrize("case", ["failed_wait", "rounding", "dropped"])
def test_pool(checker, case):
    r = subprocess.run([checker, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
