"""The library's host code driven without a GPU: fw2.cpp and setup.cpp linked
with a test double of the HIP runtime and of the device launchers
(tests/host/fake_runtime.hpp).  What is checked is which route a call takes."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_2106_11476_amd", "csrc")


@pytest.mark.parametrize("driver", ["devices_driver.cpp"])
def test_host_routes(driver, tmp_path):
    from paper_2106_11476_amd import build
    exe = str(tmp_path / "driver")
    subprocess.check_call([build.hipcc(), "-std=c++17", "-O1", "--offload-arch=gfx950", "-I", os.path.join(ROOT, "include"),
                           "-I", CSRC, "-I", HOST, os.path.join(CSRC, "fw2.cpp"), os.path.join(CSRC, "setup.cpp"),
                           os.path.join(HOST, driver), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert ": 0 failed" in r.stdout
