"""The runtime at the end of device memory (CPU only): the host sources linked
with stand-ins for the HIP runtime and the kernel launchers
(tests/host/memory_driver.cpp) that count allocations, fail them one by one, and
report a launch that is given a null or a freed buffer."""
import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_07967_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not os.path.exists(CLANG), reason="ROCm clang not installed")


@pytest.fixture(scope="module")
def driver():
    td = tempfile.mkdtemp(prefix="fgs_memory_")
    objs = []
    for src in (*(os.path.join(CSRC, f) for f in ("runtime.cpp", "pipeline.cpp", "server.cpp")),
                os.path.join(ROOT, "tests", "host", "memory_driver.cpp")):
        obj = os.path.join(td, os.path.basename(src) + ".o")
        subprocess.run([CLANG, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-O1",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", src, "-o", obj], check=True)
        objs.append(obj)
    exe = os.path.join(td, "memory_driver")
    subprocess.run([CLANG, *objs, "-lpthread", "-o", exe], check=True)
    yield exe
    shutil.rmtree(td, ignore_errors=True)


@pytest.mark.parametrize("what", ["growth", "spare", "threads"])
def test_memory(driver, what):
    r = subprocess.run([driver, what], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "memory ok" in r.stdout, r.stdout + r.stderr[:4000]
