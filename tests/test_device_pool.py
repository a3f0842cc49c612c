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


@pytest.mark.parametrize("case", ["failed_wait", "rounding", "dropped", "most_kept", "ageing",
                                  "full_device", "given_back"])
def test_pool(checker, case):
    r = subprocess.run([checker, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_binding_tries_again_without_the_kept_memory(monkeypatch):
    """A torch allocation of the binding that finds the device full."""
    import torch
    from paper_2604_18886_amd import mfmg
    calls = []

    def make(n, fails):
        calls.append("make")
        if calls.count("make") <= fails:
            raise torch.cuda.OutOfMemoryError("full")
        return n

    monkeypatch.setattr(mfmg, "release_memory", lambda: calls.append("release"))
    assert mfmg._new(make, 3, fails=1) == 3 and calls == ["make", "release", "make"]
    calls.clear()
    with pytest.raises(torch.cuda.OutOfMemoryError):
        mfmg._new(make, 3, fails=2)
