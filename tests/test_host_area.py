"""The unit kernel's clipped area by integration, compiled for the host, against polygon clipping in
exact rationals: pieces of small, large, flat and needle-shaped triangles, on and off the voxel
planes, and the pieces of one triangle against its whole area.

A piece that the integration takes is at least 2^-20 M voxel^2 (M: the triangle's extent in voxels,
plus 2) and off by less than M 2^-44; smaller ones take the other routine, good to 1e-10 of the whole.
Both are scaled by the FP32 whole area and rounded to FP32 (2e-7), and exact zeros are zeros."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import brute

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def area(tmp_path_factory):
    cxx = shutil.which("g++")
    inc = "/opt/rocm/include"
    if cxx is None or not os.path.isdir(inc):
        pytest.skip("needs g++ and the HIP headers")
    out = tmp_path_factory.mktemp("area") / "libhostarea.so"
    subprocess.run([cxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", f"-I{inc}",
                    f"-I{ROOT}/paper_2604_13191_amd/csrc", f"-I{ROOT}/include",
                    os.path.join(ROOT, "tests", "host_area.cpp"), "-o", str(out)], check=True)
    L = ctypes.CDLL(str(out))
    for f in (L.ha_area, L.ha_small):
        f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
        f.restype = ctypes.c_float

    def call(f, q, v, sb):
        e0, e1 = (q[1] - q[0]).astype(float), (q[2] - q[0]).astype(float)
        n = np.cross(e0, e1)
        l = np.linalg.norm(n)
        d = np.append(n / l if l else n, l / float(1 << sb) ** 2).astype(np.float32)
        q9, v3 = np.ascontiguousarray(q.reshape(9), np.int32), np.ascontiguousarray(v, np.int32)
        return f(q9.ctypes.data, v3.ctypes.data, sb, d.ctypes.data)

    return lambda q, v, sb: call(L.ha_area, q, v, sb), lambda q, v, sb: call(L.ha_small, q, v, sb)


def _triangle(rng, mode, s):
    if mode == 0:
        q = rng.integers(0, 8 * s, size=(3, 3))                                # generic
    elif mode == 1:
        q = rng.integers(0, 2 * s, size=(3, 3)) + 2 * s                        # about a voxel
    elif mode == 2:
        q = rng.integers(0, 16, size=(3, 3)) * (s // 2)                        # half-voxel lattice
    elif mode == 3:
        q = rng.integers(0, 8 * s, size=(3, 3))
        q[:, rng.integers(0, 3)] = rng.integers(1, 7) * s                      # flat on a voxel plane
    elif mode == 4:
        q = rng.integers(0, 8 * s, size=(1, 3)) + np.zeros((3, 1), np.int64)
        q[1] += rng.integers(-3 * s, 3 * s, size=3)
        q[2] = q[1] + rng.integers(-1, 2, size=3)                              # needle
    elif mode == 5:
        q = rng.integers(0, 2 * s, size=(3, 3)) + 3 * s
        q[:, rng.integers(0, 3)] += np.arange(3) % 2                           # nearly flat
    else:
        q = rng.integers(-40 * s, 48 * s, size=(3, 3))                         # much larger than the grid
    return q.astype(np.int64)


@pytest.mark.parametrize("sb", [3, 4, 11, 17])
def test_pieces(area, sb):
    rng = np.random.default_rng(sb)
    s, taken, zeros = 1 << sb, 0, 0
    for i in range(420):
        q = _triangle(rng, i % 7, s)
        n = np.cross(q[1] - q[0], q[2] - q[0])
        whole = 0.5 * float(np.linalg.norm(n.astype(float))) / s ** 2
        M = float((q.max(0) - q.min(0)).max()) / s + 2.0
        lo = np.maximum(-((-q.min(0)) // s) - 1, 0)
        hi = np.minimum(q.max(0) // s, 7)
        if whole == 0.0 or (hi < lo).any():
            continue
        for _ in range(3):
            v = np.array([int(rng.integers(a, b + 1)) for a, b in zip(lo, hi)], np.int64)
            ref = brute.tri_area(q, [int(x) * s for x in v], s)
            got = area[0](q, v, sb)
            if ref == 0.0:
                zeros += 1
                assert got == 0.0, (q.tolist(), v.tolist(), got)
            else:
                taken += 1
                small = ref < 2.0 ** -19 * M               # (a projection keeps more than half)
                tol = 2e-7 * ref + (1e-10 * whole if small else 2.0 ** -44 * M)
                assert abs(got - ref) <= tol, (q.tolist(), v.tolist(), got, ref)
    assert taken > 300 and zeros > 20


@pytest.mark.parametrize("sb", [4, 12])
def test_pieces_make_the_whole(area, sb):
    rng = np.random.default_rng(10 + sb)
    s = 1 << sb
    for i in range(60):
        q = _triangle(rng, (0, 1, 2, 3, 5)[i % 5], s)
        e = np.cross((q[1] - q[0]).astype(float), (q[2] - q[0]).astype(float))
        whole = 0.5 * np.linalg.norm(e) / s ** 2
        lo, hi = np.maximum(-((-q.min(0)) // s) - 1, 0), q.max(0) // s
        total = sum(area[0](q, np.array([x, y, z]), sb) for x in range(lo[0], hi[0] + 1)
                    for y in range(lo[1], hi[1] + 1) for z in range(lo[2], hi[2] + 1))
        assert abs(total - whole) <= 2e-7 * whole, (q.tolist(), total, whole)


@pytest.mark.parametrize("sb", [11, 13, 17])
def test_both_routines_round_alike(area, sb):
    """A piece close to a boundary between two floats takes the other routine: the last bits agree."""
    rng = np.random.default_rng(20 + sb)
    s, taken = 1 << sb, 0
    for i in range(9000):
        q = _triangle(rng, (0, 1, 2, 5)[i % 4], s)
        lo, hi = np.maximum(-((-q.min(0)) // s) - 1, 0), q.max(0) // s
        if not np.cross(q[1] - q[0], q[2] - q[0]).any():
            continue
        v = np.array([int(rng.integers(a, b + 1)) for a, b in zip(lo, hi)], np.int64)
        got, ref = area[0](q, v, sb), area[1](q, v, sb)
        taken += ref > 0.0
        assert got == ref, (q.tolist(), v.tolist(), got, ref)
    assert taken > 1500


@pytest.mark.parametrize("q, v, sb", [
    ([22788, 26864, 18218, 16626, 22992, 18199, 19711, 28176, 21545], [2, 3, 2], 13),
    ([5831, 5745, 7748, 4542, 8139, 5147, 4886, 5213, 7853], [2, 2, 3], 11),
    ([25191, 21514, 30530, 20927, 20759, 30521, 18711, 20549, 27379], [3, 2, 3], 13),
    ([7172, 4848, 6069, 7144, 4665, 6694, 7843, 4774, 6985], [3, 2, 3], 11),
    ([7128, 4208, 6212, 6797, 5036, 4460, 4797, 4482, 4774], [2, 2, 2], 11),
    ([7938, 4880, 7426, 4994, 7124, 8113, 7524, 6080, 7828], [2, 3, 3], 11)])
def test_scaled_by_the_same_float(area, q, v, sb):
    """Pieces whose area times the doubled area lies so near a float's boundary that the product with any
    other double than that float rounds the other way."""
    q, v = np.array(q, np.int64).reshape(3, 3), np.array(v, np.int64)
    assert area[0](q, v, sb) == area[1](q, v, sb)
