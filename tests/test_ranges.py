"""The bounds that the kernels' unchecked inner loops rely on, evaluated on the
CPU from the very functions that the kernels inline."""
import ctypes
import math
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def ranges(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("ranges") / "ranges.so")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc, "-std=c++17", "-O2", "-fPIC", "-shared", "--offload-host-only", "-o", out,
                           os.path.join(HERE, "ranges_host.hip")])
    L = ctypes.CDLL(out)
    f, i = ctypes.c_float, ctypes.c_int
    L.cell_range_of.argtypes = [f, f, f, f, i, i, i, ctypes.POINTER(i), ctypes.POINTER(i)]
    L.cell_range_of.restype = None
    L.sample_beyond_of.argtypes = [i, i, f, f, f]
    L.sample_beyond_of.restype = i
    L.clip_margin_of.argtypes = [f]
    L.clip_margin_of.restype = f
    return L


def _cells(L, X0, Y0, eX, eY, nx, ny):
    first, last = ctypes.c_int(), ctypes.c_int()
    L.cell_range_of(X0, Y0, eX, eY, nx, ny, 4, ctypes.byref(first), ctypes.byref(last))
    return first.value, last.value


# steps along an axis carry what rounding leaves of the cosine of a right angle
TINY = [0.0, 6e-17, -6e-17, 4.4e-8, -4.4e-8, 1e-20]


@pytest.mark.parametrize("shape", [(1, 1), (1, 70), (70, 1), (2, 2), (2, 70), (70, 2), (3, 3), (3, 70), (40, 50)])
def test_unchecked_samples_lie_inside(ranges, shape):
    """Every sample that is read without bounds checks has its four pixels in
    the image, for rays along an axis, steep and oblique ones, through pixel
    centres, edges and far-off anchors."""
    ny, nx = shape
    rng = np.random.default_rng(1)
    rays = [(x, y, ex, ey) for t in TINY for s in (0.5, -0.5, 1.0)
            for x, y, ex, ey in ([(0.5 * nx, v, s, t) for v in (0.0, 1e-3, -1e-3, 0.5 * (ny - 1), ny - 1.0, ny - 0.5)] +
                                 [(v, 0.5 * ny, t, s) for v in (0.0, 1e-3, -1e-3, 0.5 * (nx - 1), nx - 1.0, nx - 0.5)])]
    for _ in range(400):
        a, r = rng.uniform(0, 2 * math.pi), rng.uniform(-1.5, 1.5) * max(nx, ny)
        far = rng.choice([0.0, 1e3, 6e5, 3e6])   # an image far off the axis of rotation
        rays.append((0.5 * nx + far - r * math.sin(a), 0.5 * ny + r * math.cos(a), 0.5 * math.cos(a), 0.5 * math.sin(a)))
        rays.append((0.5 * nx - r * math.sin(a), 0.5 * ny - far, 0.5 * math.cos(a), 0.5 * math.sin(a)))
    seen = 0
    for ray in rays:
        X0, Y0, eX, eY = (np.float32(v) for v in ray)
        first, last = _cells(ranges, X0, Y0, eX, eY, nx, ny)
        if first > last:
            continue
        m = np.unique(np.clip(np.concatenate([first + np.arange(4), last - np.arange(4),
                                              np.linspace(first, last, 50).round()]), first, last))
        # the kernel's fused multiply-add rounds once
        X = (m * np.float64(eX) + np.float64(X0)).astype(np.float32)
        Y = (m * np.float64(eY) + np.float64(Y0)).astype(np.float32)
        assert X.min() >= 0 and Y.min() >= 0 and X.max() < nx - 1 and Y.max() < ny - 1, (ray, first, last)
        seen += 1
    assert seen == 0 if min(shape) < 2 else seen > 0


@pytest.mark.parametrize("m,last", [(0, 0), (5, 700), (-300, 4), (1 << 22, (1 << 22) + 90), (-(1 << 22), 1 << 22)])
@pytest.mark.parametrize("step", [0.5, 1.0, 1e-3, 3e-9, 1e-12, 1e-19])
def test_sample_beyond_stays_in_range(ranges, m, last, step):
    """The guess at where a ray leaves a slab lies in m + 1 .. last + 1, so that
    the search from it takes a bounded number of steps, however slowly the ray
    advances."""
    for sign in (1.0, -1.0):
        rate = float(np.float32(1.0) / np.float32(sign * step))
        for gap in (0.0, 0.25, 6.9, -1e-3):
            n = ranges.sample_beyond_of(m, last, 100.0 + sign * gap, 100.0, rate)
            assert m + 1 <= n <= max(last, m) + 1
            if gap > 0 and gap / step < 1e6:
                assert abs(min(m + gap / step, last + 1) - n) <= 1 + 1e-5 * gap / step


@pytest.mark.parametrize("e_max", [1e-3, 0.3, 0.5, 1.0, 49.0, 51.0, 99.0, 101.0, 150.0, 1e4])
def test_clip_margin_is_less_than_a_voxel(ranges, e_max):
    """The accumulator's halo is one voxel beyond the clip box, whatever the
    sampling step; within it the margin is 0.01 step or half a voxel."""
    margin = ranges.clip_margin_of(1.0 / e_max)
    assert margin * e_max <= 0.5 * (1 + 1e-6)
    assert margin == pytest.approx(min(0.01, 0.5 / e_max))
