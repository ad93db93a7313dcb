"""The pool of kept memory on the CPU, over HIP stand-ins that can be told to
fail: what is kept is neither dropped nor lost, whatever call is refused."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_14266_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("pool") / "pool_driver")
    cmd = [gxx, "-O1", "-g", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-x", "c++", os.path.join(CSRC, "ba_mem.hip"),
           os.path.join(ROOT, "tests", "pool_driver.cpp"), "-pthread", "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


@pytest.mark.parametrize("scenario", ["refused", "unreleased", "lack", "no_host_memory", "held"])
def test_pool(driver, scenario):
    r = subprocess.run([driver, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
