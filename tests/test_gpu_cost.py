"""Costs that calls have on the GPU relative to each other, where a choice of
kernel or a short cut is meant to keep them so.  The bounds leave a factor of
two or more to both sides."""
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
