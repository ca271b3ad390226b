"""quotient(): the correctly rounded a / d by a reciprocal of a few units' error and the exact remainder,
compiled for the host, against the division itself: bit for bit, over all sizes of integers below 2^26
and the powers of two that the callers scale by."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def differ(tmp_path_factory):
    cxx = shutil.which("g++")
    inc = "/opt/rocm/include"
    if cxx is None or not os.path.isdir(inc):
        pytest.skip("needs g++ and the HIP headers")
    out = tmp_path_factory.mktemp("quotient") / "libhostquotient.so"
    subprocess.run([cxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", f"-I{inc}",
                    f"-I{ROOT}/paper_2604_13191_amd/csrc", f"-I{ROOT}/include",
                    os.path.join(ROOT, "tests", "host_quotient.cpp"), "-o", str(out)], check=True)
    f = ctypes.CDLL(str(out)).hq_differ
    f.argtypes, f.restype = [ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_uint], ctypes.c_long
    return f


@pytest.mark.parametrize("off", [0, 1, 8])
@pytest.mark.parametrize("scale", [0, -3, -23])
def test_quotient_is_the_division(differ, off, scale):
    assert differ(1_000_000, off, scale, 7 * off - scale) == 0
