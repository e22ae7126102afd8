"""The render server's device work is ordered (CPU only): the host sources are
compiled for the host and linked with stand-ins for the HIP runtime and the
kernel launchers that keep vector clocks (tests/host/server_order_driver.cpp).
A slot whose request was refused takes part in the next shared first half,
which writes its buffers from another slot's stream; with many Gaussians the
refused request's depth order is eight launches, with few it is one."""
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
    td = tempfile.mkdtemp(prefix="fgs_order_")
    objs = []
    for src in (*(os.path.join(CSRC, f) for f in ("runtime.cpp", "pipeline.cpp", "server.cpp")),
                os.path.join(ROOT, "tests", "host", "server_order_driver.cpp")):
        obj = os.path.join(td, os.path.basename(src) + ".o")
        subprocess.run([CLANG, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-O1",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", src, "-o", obj], check=True)
        objs.append(obj)
    exe = os.path.join(td, "server_order_driver")
    subprocess.run([CLANG, *objs, "-lpthread", "-o", exe], check=True)
    yield exe
    shutil.rmtree(td, ignore_errors=True)


@pytest.mark.parametrize("P", [100_000, 1_000])
def test_a_refused_slot_joins_a_shared_first_half(driver, P):
    r = subprocess.run([driver, str(P)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "order ok" in r.stdout, r.stdout + r.stderr
