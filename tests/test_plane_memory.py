"""The plane pass's memory is optional (no GPU needed): host paths of libgps.so against a
HIP runtime of its own (tests/host_alloc/fake_hip.h) whose device memory has a limit."""
import os
import shutil
import subprocess
import tempfile

import pytest

from paper_1509_00680_amd import gps

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
HIPCC = os.environ.get("HIPCC", os.path.join(ROCM, "bin", "hipcc"))
CSRC = os.path.join(ROOT, "paper_1509_00680_amd", "csrc")


def run_host(source, internal=False):
    """Compiles tests/host_alloc/<source> against the library and runs it; internal: with the
    library's own headers (host side only)."""
    d = tempfile.mkdtemp(prefix="gps_host_")
    try:
        exe = os.path.join(d, "host")
        lib = os.path.dirname(gps.load()._name)
        obj = os.path.join(d, "host.o")
        cc = [HIPCC, "--offload-host-only", "-I", CSRC] if internal else ["g++"]
        r = subprocess.run(cc + ["-std=c++17", "-O1", "-g", "-fPIE", "-D__HIP_PLATFORM_AMD__",
                                 "-I", os.path.join(ROCM, "include"),
                                 "-I", os.path.join(ROOT, "include"), "-c",
                                 os.path.join(HERE, "host_alloc", source), "-o", obj],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        r = subprocess.run(["g++", "-rdynamic", obj, "-o", exe, "-L", lib, "-lgps",
                            "-Wl,-rpath," + lib, "-Wl,-rpath," + os.path.join(ROCM, "lib"),
                            "-L", os.path.join(ROCM, "lib")], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        return subprocess.run([exe], capture_output=True, text=True, timeout=300)
    finally:
        shutil.rmtree(d, ignore_errors=True)


needs_host = pytest.mark.skipif(shutil.which("g++") is None or
                                not os.path.exists(os.path.join(ROCM, "include", "hip")),
                                reason="needs g++ and the HIP headers")


@needs_host
def test_calls_run_where_they_ran_without_the_plane_pass():
    r = run_host("plane_memory.cpp")
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    assert " 0 failures" in r.stdout


@needs_host
@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_modes_beside_the_plane_pass():
    r = run_host("plane_modes.cpp", internal=True)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    assert " 0 failures" in r.stdout
