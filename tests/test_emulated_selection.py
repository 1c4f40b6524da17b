"""The volume-preserving selection's kernels on the CPU (tests/host/emulated_gpu.hpp), under
an address sanitizer, against a sort."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_1711_01365_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not os.path.exists(CLANG), reason="ROCm's clang not installed")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("emulated")
    for name in os.listdir(CSRC):
        if name.endswith(".hpp") or name == "mbo_volume.hip":
            with open(os.path.join(CSRC, name)) as f:
                text = f.read()
            # dynamic shared memory: not used by the kernels run here
            text = text.replace("extern __shared__ __align__(16) unsigned char smem_raw[];",
                                "alignas(16) static unsigned char smem_raw[1];")
            (d / name).write_text(text)
    flags = ["-std=c++17", "-O1", "-g", "-w", "-D__HIP_PLATFORM_AMD__", "-fsanitize=address", "-ffp-contract=off",
             "-I", str(d), "-I", HERE, "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include")]
    jobs = [(["-include", "emulated_gpu.hpp", "-x", "c++", str(d / "mbo_volume.hip")], "volume.o"),
            ([os.path.join(HERE, "emulated_gpu.cpp")], "emulated.o"),
            ([os.path.join(HERE, "selection_driver.cpp")], "driver.o")]
    running = [subprocess.Popen([CLANG] + flags + src + ["-c", "-o", str(d / obj)], stderr=subprocess.PIPE, text=True)
               for src, obj in jobs]
    for p in running:
        err = p.communicate()[1]
        assert p.returncode == 0, err[-3000:]
    exe = str(d / "selection_driver")
    subprocess.run([CLANG, "-fsanitize=address", "-o", exe] + [str(d / o) for _, o in jobs], check=True)
    return exe


@pytest.mark.parametrize("seed", range(4))
def test_selection_is_the_sorts(driver, seed):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0")
    r = subprocess.run([driver, str(seed), "25"], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr[-3000:]
