"""The autotuner's choices (no GPU): csrc/tune.cpp built with a model of the device (tests/tune/tune_main.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def tuner(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("g++ or the HIP headers not found")
    exe = str(tmp_path_factory.mktemp("tune") / "tune_host")
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{ROOT}/include", "-o", exe,
           os.path.join(HERE, "tune", "tune_main.cpp"), os.path.join(ROOT, "paper_2109_05072_amd", "csrc", "tune.cpp")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("what", ["default", "source", "cache", "once"])
def test_tuner(tuner, tmp_path, what):
    r = subprocess.run([tuner, what], capture_output=True, text=True, cwd=tmp_path, timeout=60,
                       env={k: v for k, v in os.environ.items() if k != "MFHEX_TUNE_CACHE"})
    assert r.returncode == 0 and "OK" in r.stdout, r.stdout + r.stderr
