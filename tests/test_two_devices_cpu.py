"""What the library keeps per device, without a GPU: tests/host/two_devices.cpp stands in for the HIP
calls, runs the library's launchers and allocations as on two devices, and checks what each was asked."""
import os
import shutil
import subprocess

import pytest

from paper_2310_16238_amd import coxmi

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2310_16238_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("needs g++ and HIP headers")
    coxmi.lib()
    exe = str(tmp_path_factory.mktemp("host") / "two_devices")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I",
           os.path.join(PKG, "csrc"), "-I", "/opt/rocm/include", os.path.join(ROOT, "tests", "host", "two_devices.cpp"),
           "-L", PKG, "-l:libcoxmi.so", "-Wl,-rpath," + PKG, "-Wl,-rpath-link,/opt/rocm/lib", "-lpthread", "-o", exe]
    subprocess.run(cmd, check=True, timeout=300)
    return exe


@pytest.mark.parametrize("what", ["lds", "memory"])
def test_state_is_kept_per_device(program, what):
    r = subprocess.run([program, what], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout + r.stderr
