"""The library's host code driven without a GPU: fw2.cpp and setup.cpp linked
with a test double of the HIP runtime and of the device launchers
(tests/host/fake_runtime.hpp).  What is checked is which route a call takes."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_2106_11476_amd", "csrc")


def _compile(*args):
    from paper_2106_11476_amd import build
    subprocess.check_call([build.hipcc(), "--cuda-host-only", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
                           "-I", CSRC, "-I", HOST] + list(args))


@pytest.fixture(scope="module")
def host_objects(tmp_path_factory):
    """The library's host code, compiled once for all drivers."""
    out = tmp_path_factory.mktemp("host")
    objects = []
    for name in ("fw2.cpp", "setup.cpp"):
        objects.append(str(out / (name + ".o")))
        _compile("-c", os.path.join(CSRC, name), "-o", objects[-1])
    return objects


@pytest.mark.parametrize("driver", ["devices_driver.cpp", "workspace_driver.cpp", "sources_driver.cpp",
                                    "tiles_driver.cpp", "limits_driver.cpp", "bands_driver.cpp"])
def test_host_routes(driver, host_objects, tmp_path):
    exe = str(tmp_path / "driver")
    _compile("-c", os.path.join(HOST, driver), "-o", exe + ".o")
    _compile(exe + ".o", *host_objects, "-o", exe)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert ": 0 failed" in r.stdout


@pytest.mark.parametrize("shape,L", [((128, 128), 2), ((384, 260), 4), ((1024, 1024), 2), ((2400, 1500), 2), ((300, 200), 6)])
def test_served_requests_hold_one_state_block(shape, L):
    """The bytes a served request is admitted by: state and medium once (a
    request stepped in a batch has no use for a second state block)."""
    import numpy as np

    import workloads as W
    from paper_2106_11476_amd import fw2, serve
    prob = W.homogeneous(shape, L=L)
    prob.rcv_idx = np.zeros(0, np.int64)
    stride = (shape[0] + 8 + 63) // 64 * 64 * (shape[1] + 8) * 4
    arrays = 1 + 2 + 4 * L + 3
    assert arrays * stride <= fw2.workspace_bytes(prob) < arrays * stride + (1 << 16)
    assert serve.footprint_bytes(prob, 10) - fw2.workspace_bytes(prob) < 1 << 16


def test_the_autotuner_times_each_kernel_once():
    """Its default candidates ask for the two tiles that the batched kernels
    have: 64 x 8, and 64 x 16 for more than 256 x 4."""
    import inspect

    from paper_2106_11476_amd import serve
    tiles = inspect.signature(serve.autotune_tile).parameters["candidates"].default
    rows = [16 if r >= (16 if c == 64 else 5) else 8 for c, r in tiles]
    assert sorted(rows) == [8, 16]
