"""The host side of the C ABI (mbo_api.cpp) on a fake HIP runtime, without a GPU: device
memory that is refused, pinned buffers, and the streams that work goes to (tests/host)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_1711_01365_amd", "csrc")
ROCM = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(ROCM, "hip", "hip_runtime.h")),
                                reason="HIP headers not installed")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "plan_driver")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", "-I", ROCM, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", HERE,
           os.path.join(CSRC, "mbo_api.cpp"), os.path.join(HERE, "fake_runtime.cpp"),
           os.path.join(HERE, "plan_driver.cpp"), "-pthread", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("scenario", ["set_tau_2d", "set_tau_3d", "volume_memory", "adjoint_memory",
                                      "surface_memory", "pinned_buffers", "field_word"])
def test_scenario(driver, scenario):
    r = subprocess.run([driver, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr[-3000:]
