"""The bookkeeping of the handle's kept scratch blocks (scratch.hpp) without a
GPU, against a stand-in for the runtime calls it makes."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    out = str(tmp_path_factory.mktemp("scratch") / "scratch")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                        "-I", os.path.join(HERE, "scratch_stub"),
                        os.path.join(HERE, "scratch_stub", "main.cpp"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


@pytest.mark.parametrize("what", ["errors", "bounds", "optional", "host_memory"])
def test_scratch(exe, what):
    r = subprocess.run([exe, what], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr[-2000:]
