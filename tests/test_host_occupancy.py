"""A capsule's sub-cells, compiled for the host, bit for bit against the exact test of every sub-cell:
segments from one end of the grid to the other on grids of 2^10 to 2^17 voxels an axis, whose distances
from a voxel are differences of numbers up to 2^40 sub-cells squared, and short ones."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _fma():
    try:
        with open("/proc/cpuinfo") as f:
            return " fma " in f.read()
    except OSError:
        return False


@pytest.fixture(scope="module", params=["separate", "fused"])
def masks(request, tmp_path_factory):
    """Products and sums rounded apart, and fused where the compiler may, as on the device."""
    if request.param == "fused" and not _fma():
        pytest.skip("no fused multiply-add")
    cxx = shutil.which("g++")
    inc = "/opt/rocm/include"
    if cxx is None or not os.path.isdir(inc):
        pytest.skip("needs g++ and the HIP headers")
    out = tmp_path_factory.mktemp("occ") / "libhostocc.so"
    subprocess.run([cxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", f"-I{inc}",
                    *(["-mfma"] if request.param == "fused" else []),
                    f"-I{ROOT}/paper_2604_13191_amd/csrc", f"-I{ROOT}/include",
                    os.path.join(ROOT, "tests", "host_occupancy.cpp"), "-o", str(out)], check=True)
    L = ctypes.CDLL(str(out))
    P, I = ctypes.c_void_p, ctypes.c_int
    L.ho_wrong.argtypes = [P, P, I, ctypes.c_int64, ctypes.POINTER(I)]
    L.ho_touch.argtypes = [P, P, I, ctypes.c_int64]

    def wrong(r, v, sb, rho):
        """(wrong bits, exact hits) of a segment [6] in a voxel, or None where it does not touch it"""
        r, v = np.ascontiguousarray(r, np.int32), np.ascontiguousarray(v, np.int64)
        if not L.ho_touch(r.ctypes.data, v.ctypes.data, sb, rho):
            return None
        n = ctypes.c_int()
        return L.ho_wrong(r.ctypes.data, v.ctypes.data, sb, rho, ctypes.byref(n)), n.value

    return wrong


@pytest.mark.parametrize("r, v, log2, rho, hits", [
    ([0, 4194448, 4194561, 8388607, 4194448, 4194560], [32767, 16384, 16384], 15, 128, 241),
    ([3, 4194376, 4194433, 8388603, 4194376, 4194432], [65535, 32768, 32768], 16, 64, 241),
    ([968699, 1884381, 5921476, 8324469, 1884359, 5921476], [124845, 29443, 92523], 17, 32, None)])
def test_known(masks, r, v, log2, rho, hits):
    bad, n = masks(r, v, 23 - log2, rho)
    assert bad == 0 and (hits is None or n == hits), (bad, n)


def _segment(rng, mode, s):
    """A segment's ends (lattice units)."""
    far = 1 << 23
    a, b = rng.integers(0, far, size=3), rng.integers(0, far, size=3)
    ax = int(rng.integers(0, 3))
    if mode == 0:                                              # across the grid, nearly along an axis
        b = a + rng.integers(-2, 3, size=3)
        a[ax], b[ax] = rng.integers(0, 8), far - rng.integers(0, 8)
    elif mode == 1:                                            # the same with slopes up to 1e-4
        b = a + rng.integers(-far // 10000, far // 10000 + 1, size=3)
        a[ax], b[ax] = rng.integers(0, 8), far - rng.integers(0, 8)
    elif mode == 2:                                            # along a diagonal, from far outside
        d = rng.choice([-1, 1], size=3) * (far - rng.integers(0, 4, size=3))
        a = np.where(d > 0, 0, far) + rng.integers(-8, 9, size=3)
        b = a + d
    elif mode == 3:                                            # on the corners and centres of sub-cells
        q = max(s // 16, 1)
        a, b = a // q * q, b // q * q
        b[ax] = a[ax]
    elif mode == 4:                                            # a few voxels long
        b = a + rng.integers(-3 * s, 3 * s + 1, size=3)
    return np.concatenate([a, b]).astype(np.int64)


@pytest.mark.parametrize("log2", range(10, 18))
def test_exact(masks, log2):
    rng = np.random.default_rng(log2)
    sb = 23 - log2
    s, taken, hits = 1 << sb, 0, 0
    for i in range(1500):
        r = _segment(rng, i % 5, s)
        rho = int(rng.choice([0, s // 8, s // 2, s // 2 + 1, 2 * s + 3]))
        for _ in range(10):
            t = rng.choice([rng.random(), 1.0 - 1e-4 * rng.random()])       # often near the far end
            p = r[:3] + t * (r[3:] - r[:3]) + rng.uniform(-1.0, 1.0, size=3) * (rho + s)
            v = np.floor(p / s).astype(np.int64)
            if (v < 0).any() or (v >= 1 << log2).any():
                continue
            got = masks(r, v, sb, rho)
            if got is None:
                continue
            taken, hits = taken + 1, hits + got[1]
            assert got[0] == 0, (r.tolist(), v.tolist(), rho, got)
    assert taken > 4000 and hits > 100 * taken
