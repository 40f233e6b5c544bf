"""Costs that calls have on the GPU relative to each other, where a choice of
kernel or a short cut is meant to keep them so.  The bounds lie well
between what is meant and what is not."""
import math
import time

import pytest
import torch

import gpu_common as gc
from gpu_common import say

pytestmark = pytest.mark.gpu

DEG = math.pi / 180


@pytest.fixture(scope="module")
def ph():
    gc.device()
    import paper_1904_13342_amd as ph
    return ph


def _us(call):
    """Microseconds of a call among others, the least of five runs."""
    call()
    torch.cuda.synchronize()
    best = math.inf
    for _ in range(5):
        t = time.perf_counter()
        for _ in range(10):
            call()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / 10)
    return 1e6 * best


@pytest.mark.parametrize("fan", [False, True])
def test_project_2d_narrow_detector(ph, fan):
    """The same number of rays costs alike in views of one bin and of sixty."""
    src = dict(sid=750.0, sdd=1200.0) if fan else {}
    A = ph.project_fan2d if fan else ph.project_par2d
    img = torch.rand((256, 256), device=gc.device())
    us = {}
    for nu, views in ((1, 36000), (60, 600)):
        g = ph.geom2d((256, 256), (1.0, 1.0), nu, 1.0, views, 360 * DEG, **src)
        rv = ph.ray_vectors_2d(g)
        us[nu] = _us(lambda: A(g, rv, img))
    say(f"[cost] A, 36000 rays: {us}")
    assert us[1] < 5 * us[60]


@pytest.mark.parametrize("beam,detector", [("par", "flat"), ("fan", "flat"), ("fan", "curved")])
def test_transposes_2d_of_zeros(ph, beam, detector):
    """Rays and pixels of zeros are passed over: zeros, and a single value, cost
    A^T, and B^T by runs, little more than the loads (B^T 0.3 to 0.5 of what dense
    data costs, A^T less)."""
    src = dict(sid=750.0, sdd=1200.0) if beam == "fan" else {}
    n, nu, views = 512, 725, 300
    g = ph.geom2d((n, n), (0.5, 0.5), nu, 1.0 if beam == "fan" else 0.6, views, 360 * DEG, detector=detector, **src)
    rv, dev = ph.ray_vectors_2d(g), gc.device()
    for name, shape in (("project_adjoint", (views, nu)), ("backproject_adjoint", (n, n))):
        op = getattr(ph, f"{name}_{beam}2d")
        dense, zero = torch.rand(shape, device=dev) + 0.5, torch.zeros(shape, device=dev)
        one = zero.clone()
        one[shape[0] // 2, shape[1] // 3] = 1.0
        us = [_us(lambda: op(g, rv, x)) for x in (dense, zero, one)]
        say(f"[cost] {name} {beam} {detector}: dense, zeros, one value {us}")
        assert max(us[1:]) < 0.7 * us[0]


def _device_us(call):
    """Microseconds of a call on the device: twenty in a captured graph."""
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(20):
            call()
    graph.replay()
    torch.cuda.synchronize()
    best = math.inf
    for _ in range(5):
        t = time.perf_counter()
        graph.replay()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / 20)
    return 1e6 * best


@pytest.mark.parametrize("n", [64, 128])
def test_backproject_2d_small_parallel(ph, n):
    """A small parallel item costs no more than a fan of the same size, whose
    coordinates are the dearer ones: it is not staged by a few workgroups."""
    us = {}
    for beam, src in (("par", {}), ("fan", dict(sid=750.0, sdd=1200.0))):
        g = ph.geom2d((n, n), (1.0, 1.0), 2 * n, 1.0, 360, 360 * DEG, **src)
        rv = ph.ray_vectors_2d(g)
        p, out = torch.rand((360, 2 * n), device=gc.device()), torch.empty((n, n), device=gc.device())
        op = getattr(ph, f"backproject_{beam}2d")
        us[beam] = _device_us(lambda: op(g, rv, p, out))
    say(f"[cost] B {n}^2, 360 views: {us}")
    assert us["par"] < 1.3 * us["fan"]


def _cone(ph, n, views):
    s = 256.0 / n
    nu = int(1.75 * n / 1.3)
    g = ph.geom3d((n, n, n), (s, s, s), (int(0.8 * nu), nu), (1.3 * s, 1.3 * s), views, 360 * DEG, 750.0, 1200.0)
    return g, ph.projection_matrices_3d(g)


def test_backproject_adjoint_cone_few_views(ph):
    """A quarter of the views costs B^T well under half: they are not dealt into
    shares of a handful of views."""
    us = {}
    x = torch.rand((190, 190, 190), device=gc.device())
    for views in (60, 240):
        g, mats = _cone(ph, 190, views)
        us[views] = _us(lambda: ph.backproject_adjoint_cone3d(g, mats, x))
    say(f"[cost] B^T 190^3: {us}")
    assert us[60] < 0.42 * us[240]


def test_backproject_cone_between_waves_and_bricks(ph):
    """160^3 costs no more than 176^3, which goes in bricks."""
    us = {}
    for n in (160, 176):
        g, mats = _cone(ph, n, 60)
        p = torch.rand((60,) + tuple(g.det_shape), device=gc.device())
        us[n] = _us(lambda: ph.backproject_cone3d(g, mats, p))
    say(f"[cost] B: {us}")
    assert us[160] < 1.12 * us[176]


@pytest.mark.parametrize("beam", ["par", "fan"])
def test_project_adjoint_2d_small_images(ph, beam):
    """32^2 costs A^T well under what 128^2 does, with sixteen times the pixels:
    its views are not one long chain to each of a few waves."""
    src = dict(sid=750.0, sdd=1200.0) if beam == "fan" else {}
    us = {}
    for n in (32, 128):
        g = ph.geom2d((n, n), (1.0, 1.0), 3 * n // 2, 1.0, 500, 360 * DEG, **src)
        rv = ph.ray_vectors_2d(g)
        p, out = torch.rand((500, 3 * n // 2), device=gc.device()), torch.empty((n, n), device=gc.device())
        op = getattr(ph, f"project_adjoint_{beam}2d")
        us[n] = _device_us(lambda: op(g, rv, p, out))
    say(f"[cost] A^T, 500 {beam} views: {us}")
    assert us[32] < 0.65 * us[128]


@pytest.mark.parametrize("shape", [(1000, 30), (121, 36), (36, 121)])
def test_project_2d_thin_images(ph, shape):
    """A thin image costs A no more than a square one that is longer on its rays:
    its few slabs across are not walked by one wave."""
    us = {}
    for s in (shape, (256, 256)):
        nu = int(1.45 * max(s))
        g = ph.geom2d(s, (1.0, 1.0), nu, 1.0, 2400 * 64 // nu, 360 * DEG)
        rv = ph.ray_vectors_2d(g)
        x, out = torch.rand(s, device=gc.device()), torch.empty((g.n_proj, nu), device=gc.device())
        us[s] = _device_us(lambda: ph.project_par2d(g, rv, x, out))
    say(f"[cost] A, 153600 rays: {us}")
    assert us[shape] < 1.1 * us[(256, 256)]


def test_project_adjoint_cone_coarse_detector(ph):
    """Pixels of three voxels, a ninth of the rays, cost A^T well under a third of
    what pixels of one do."""
    us = {}
    n, s = 160, 1.6
    for d in (1.0, 3.0):
        nu = int(1.75 * n / d)
        g = ph.geom3d((n, n, n), (s, s, s), (nu, nu), (d * s, d * s), 30, 360 * DEG, 750.0, 1200.0)
        mats, p = ph.projection_matrices_3d(g), torch.rand((30, nu, nu), device=gc.device())
        us[d] = _us(lambda: ph.project_adjoint_cone3d(g, mats, p))
    say(f"[cost] A^T 160^3: {us}")
    assert us[3.0] < 0.31 * us[1.0]
