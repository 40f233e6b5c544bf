"""2D projector and back-projector where the unchecked inner loops meet the
checked ones, against the FP64 oracle: images whose border is inside every
wave's four samples, images narrower than a cell, rays along an axis, an image
far off the axis of rotation, few and many rays per wave, views in numbers
that are no multiple of a lane's four."""
import math

import numpy as np
import pytest

import gpu_common as gc
import synth
from gpu_common import as_f32, check, say, to_dev, to_np

pytestmark = pytest.mark.gpu

FAN = dict(sid=700.0, sdd=1100.0)
# kind, (ny, nx), nu, du, views, range in degrees, source, origin (y, x) or None
CASES = {
    "par_2x2": ("par2d", (2, 2), 7, 0.5, 4, 180, {}, None),
    "par_row": ("par2d", (1, 70), 80, 1.0, 5, 180, {}, None),
    "par_column": ("par2d", (70, 1), 80, 1.0, 5, 180, {}, None),
    "par_axis_aligned": ("par2d", (96, 64), 101, 1.0, 4, 360, {}, None),
    "par_one_view": ("par2d", (130, 90), 160, 1.0, 1, 180, {}, None),
    "par_63_views": ("par2d", (40, 300), 310, 1.0, 63, 180, {}, None),
    "par_off_axis": ("par2d", (60, 50), 500, 1.0, 9, 180, {}, (-180.0, 120.0)),
    "fan_65_views": ("fan2d", (127, 129), 230, 1.0, 65, 360, FAN, None),
    "fan_few_bins": ("fan2d", (100, 90), 3, 60.0, 33, 360, FAN, None),
    # slabs: 64 rays to a wave, the last wave of one ray; bins wider than the
    # widest slab; a step longer than a pixel; rays at 45 degrees
    "par_65_bins": ("par2d", (61, 83), 65, 1.3, 8, 180, {}, None),
    "par_wide_bins": ("par2d", (70, 64), 50, 1.75, 7, 180, {}, None),
    "par_very_wide_bins": ("par2d", (70, 64), 40, 2.6, 7, 180, {}, None),
    "par_diagonal": ("par2d", (200, 190), 280, 1.0, 8, 360, {}, None),
    "fan_steep": ("fan2d", (80, 300), 400, 1.2, 12, 360, dict(sid=190.0, sdd=300.0), None),
    "arc_short": ("fan2d_curved", (90, 128), 190, 1.1, 37, 220, FAN, None),
}


@pytest.fixture(scope="module")
def ph():
    gc.device()
    import paper_1904_13342_amd as ph
    return ph


@pytest.mark.parametrize("name", list(CASES))
def test_pair_2d_edges(ph, ora, name):
    kind, shape, nu, du, views, turn, src, origin = CASES[name]
    spec = synth.config("par2d_64").with_(kind=kind, vol_shape=shape, vol_spacing=(1.0, 1.0), det_shape=(nu,),
                                          det_spacing=(du,), n_proj=views, angular_range=turn * math.pi / 180,
                                          vol_origin=origin, **src)
    g = ph.from_spec(spec)
    rv, fan = ph.ray_vectors_2d(g), kind != "par2d"
    rng = np.random.default_rng(3)
    # positive values: a sum of terms that do not cancel keeps the coordinates'
    # rounding (2^-17 pixel and bin) at 1e-5 of itself
    # enough items of the same two images for the slab kernel (512 waves of
    # rays), and the two alone for the direct one
    f = as_f32(rng.uniform(0.5, 1.5, (2,) + spec.vol_shape))
    p = as_f32(rng.uniform(0.5, 1.5, (2, views, nu)))
    many = -(-512 // (-(-nu // 64) * views) // 2)
    A, B = (ph.project_fan2d, ph.backproject_fan2d) if fan else (ph.project_par2d, ph.backproject_par2d)
    say(f"[A, B 2D] {name}")
    check(to_np(A(g, rv, to_dev(f))), np.stack([ora.project(spec, v) for v in f]), "A", tol=2e-5)
    out = A(g, rv, to_dev(f).repeat(many, 1, 1))
    check(to_np(out[:2]), np.stack([ora.project(spec, v) for v in f]), "A, many items", tol=2e-5)
    assert (out.view((many, 2) + tuple(out.shape[1:])) == out[:2]).all()
    check(to_np(B(g, rv, to_dev(p))), np.stack([ora.backproject(spec, v) for v in p]), "B", tol=2e-5)


@pytest.mark.parametrize("step", [0.1, 0.7, 1.0, 1.3])
def test_project_2d_steps(ph, ora, step):
    """Sampling steps from a tenth of a pixel to more than one."""
    spec = synth.config("par2d_64").with_(vol_shape=(90, 75), vol_spacing=(1.0, 1.2), det_shape=(131,),
                                          det_spacing=(0.9,), n_proj=9, step_mm=step)
    g = ph.from_spec(spec)
    rv = ph.ray_vectors_2d(g)
    f = as_f32(np.random.default_rng(8).uniform(0.5, 1.5, spec.vol_shape))
    ref = ora.project(spec, f)
    check(to_np(ph.project_par2d(g, rv, to_dev(f))), ref, f"step {step}, direct", tol=2e-5)
    check(to_np(ph.project_par2d(g, rv, to_dev(f).repeat(20, 1, 1))[19]), ref, f"step {step}, slabs", tol=2e-5)


# kind, (ny, nx), nu, du, views, range, source, origin, items: one item and
# items in groups of two and four with one left over, by number of 16 x 16
# tiles; 32 and 64 bins to a view, and more than fit; tiles, views and waves
# with remainders; tiles off the detector
SEGMENTS = {
    "par_one": ("par2d", (45, 33), 61, 1.0, 17, 180, {}, None, 1),
    "par_64_bins": ("par2d", (45, 33), 240, 0.4, 33, 180, {}, None, 1),
    "par_too_fine": ("par2d", (30, 33), 200, 0.3, 5, 180, {}, None, 2),
    "par_groups_of_2": ("par2d", (130, 144), 150, 1.0, 31, 180, {}, None, 5),
    "par_groups_of_4": ("par2d", (257, 270), 300, 1.0, 7, 180, {}, (-140.0, -90.0), 5),
    "flat_groups_of_2": ("fan2d", (130, 144), 210, 1.7, 31, 360, FAN, None, 5),
    "flat_64_bins": ("fan2d", (257, 270), 300, 0.9, 7, 360, FAN, None, 3),
    "arc_groups_of_4": ("fan2d_curved", (257, 270), 400, 1.9, 7, 360, FAN, None, 5),
    "arc_wide_fan": ("fan2d_curved", (130, 300), 300, 2.6, 19, 360, dict(sid=210.0, sdd=300.0), None, 4),
    "arc_off_axis": ("fan2d_curved", (130, 300), 300, 2.6, 19, 360, dict(sid=260.0, sdd=420.0), (-60.0, -110.0), 4),
}


@pytest.mark.parametrize("name", list(SEGMENTS))
def test_backproject_2d_segments(ph, ora, name):
    kind, shape, nu, du, views, turn, src, origin, items = SEGMENTS[name]
    spec = synth.config("par2d_64").with_(kind=kind, vol_shape=shape, vol_spacing=(1.0, 1.0), det_shape=(nu,),
                                          det_spacing=(du,), n_proj=views, angular_range=turn * math.pi / 180,
                                          vol_origin=origin, **src)
    g = ph.from_spec(spec)
    p = as_f32(np.random.default_rng(5).uniform(0.5, 1.5, (items, views, nu)))
    B = ph.backproject_fan2d if kind != "par2d" else ph.backproject_par2d
    say(f"[B 2D segments] {name}")
    out = to_np(B(g, ph.ray_vectors_2d(g), to_dev(p)))
    for n in {0, items // 2, items - 1}:
        check(out[n], ora.backproject(spec, p[n]), f"item {n}", tol=2e-5)


@pytest.mark.parametrize("shape", [(1, 1), (1, 70), (70, 1), (2, 70), (70, 2), (3, 70)])
@pytest.mark.parametrize("kind,du", [("par2d", 1.0), ("par2d", 2.0), ("fan2d", 2.0), ("fan2d_curved", 3.0)])
def test_project_2d_thin_images(ph, ora, kind, du, shape):
    """Images of one to three rows or columns, rays along them through their
    centres (odd bins, views a quarter turn apart): no 2 x 2 cell lies inside
    the thinnest, and the two items differ, so a read past one would show."""
    spec = synth.config("par2d_64").with_(kind=kind, vol_shape=shape, vol_spacing=(1.0, 1.0), det_shape=(81,),
                                          det_spacing=(du,), n_proj=8, angular_range=2 * math.pi,
                                          **({} if kind == "par2d" else FAN))
    g = ph.from_spec(spec)
    rv = ph.ray_vectors_2d(g)
    f = as_f32(np.random.default_rng(2).uniform(0.5, 1.5, (2,) + shape) * np.array([1.0, 100.0])[:, None, None])
    A = ph.project_par2d if kind == "par2d" else ph.project_fan2d
    say(f"[A 2D] {kind} {shape} bins of {du}")
    out = to_np(A(g, rv, to_dev(f)))
    for n in range(2):
        check(out[n], ora.project(spec, f[n]), f"item {n}", tol=2e-5)


@pytest.mark.parametrize("nu,du,views", [(345, 1.4, 90), (345, 1.4, 300), (250, 1.9, 140)])
def test_project_2d_wide_slabs(ph, ora, nu, du, views):
    """The widest slabs with as many waves to a workgroup as its share of the
    LDS holds, and bins just too wide for them."""
    spec = synth.config("par2d_64").with_(vol_shape=(341, 345), vol_spacing=(1.0, 1.0), det_shape=(nu,),
                                          det_spacing=(du,), n_proj=views, angular_range=math.pi)
    g = ph.from_spec(spec)
    f = as_f32(np.random.default_rng(12).uniform(0.5, 1.5, spec.vol_shape))
    say(f"[A 2D] {nu} bins of {du}, {views} views")
    check(to_np(ph.project_par2d(g, ph.ray_vectors_2d(g), to_dev(f))), ora.project(spec, f), "A", tol=2e-5)


@pytest.mark.parametrize("du,nu", [(1.0, 380), (0.45, 860), (0.3, 1250)])
def test_backproject_2d_one_item_staged(ph, ora, du, nu):
    """One parallel item with enough tiles and views to be staged: 32 and 64
    bins to a view, and more than fit, tiles and chunks of views with
    remainders."""
    spec = synth.config("par2d_64").with_(vol_shape=(258, 270), vol_spacing=(1.0, 1.0), det_shape=(nu,),
                                          det_spacing=(du,), n_proj=107, angular_range=math.pi)
    g = ph.from_spec(spec)
    p = as_f32(np.random.default_rng(15).uniform(0.5, 1.5, (107, nu)))
    say(f"[B 2D] one item, bins of {du}")
    check(to_np(ph.backproject_par2d(g, ph.ray_vectors_2d(g), to_dev(p))), ora.backproject(spec, p), "B", tol=2e-5)
