"""The library's device-memory bookkeeping on the CPU: the host side of
primitives.hip and common.hpp with stand-ins for the HIP calls
(tests/native/memory_host_checks.cpp)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1605_01715_amd", "csrc")


@pytest.fixture(scope="module")
def checks(tmp_path_factory):
    from paper_1605_01715_amd import build as B

    cc = B.hipcc()
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("memory")
    obj, exe = str(d / "primitives.o"), str(d / "memory_host_checks")
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    subprocess.check_call([cc, "--cuda-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-g", "-Wno-unused-result", *inc,
                           "-c", os.path.join(CSRC, "primitives.hip"), "-o", obj])
    # the device code object is not there; no kernel is launched
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-g", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", *inc,
                           os.path.join(ROOT, "tests", "native", "memory_host_checks.cpp"), obj, "-no-pie",
                           "-Wl,--unresolved-symbols=ignore-in-object-files", "-lpthread", "-o", exe])
    return exe


@pytest.mark.parametrize("what", ["wait", "give", "copies", "failed_copy"])
def test_memory_bookkeeping(checks, what):
    out = subprocess.run([checks, what], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr
