"""The 2D transposes at the edges of their work split, against the FP64
oracle: bin counts around a wave's 63 strips, bins far narrower and far wider
than a pixel, images of one row, one column and one pixel, and fans whose
outer bins run across the axis the wave walks along."""
import math

import pytest

import gpu_common as gc
import synth
from gpu_common import as_f32, check, say, to_dev, to_np

pytestmark = pytest.mark.gpu

# The rays are white noise here, so a pixel's sum of n terms grows as sqrt(n)
# while FP32 sample positions (up to 2^-19 voxel off at coordinates of 64)
# move every term by up to 2^-18 of its weight: 4e-6 of the result, in terms
# that do not cancel, and up to four times that where the terms do.
TOL_AT = 2e-5

FAN = dict(sid=120.0, sdd=200.0)
# kind, (ny, nx), nu, du, views, range in degrees
CASES = {
    "par_62": ("par2d", (24, 31), 62, 0.7, 11, 180, {}),
    "par_63": ("par2d", (31, 24), 63, 0.7, 7, 180, {}),
    "par_64": ("par2d", (33, 32), 64, 0.7, 5, 360, {}),
    "par_127_fine": ("par2d", (17, 40), 127, 0.31, 8, 180, {}),
    "par_coarse": ("par2d", (64, 70), 9, 9.0, 12, 180, {}),
    "par_1_bin": ("par2d", (20, 20), 1, 4.0, 6, 180, {}),
    "par_row": ("par2d", (1, 33), 41, 1.0, 9, 180, {}),
    "par_column": ("par2d", (33, 1), 41, 1.0, 9, 180, {}),
    "par_pixel": ("par2d", (1, 1), 5, 0.6, 9, 180, {}),
    "fan_126": ("fan2d", (40, 37), 126, 0.8, 13, 360, FAN),
    "fan_wide": ("fan2d", (30, 30), 70, 9.0, 9, 360, dict(sid=40.0, sdd=60.0)),
    "arc_190": ("fan2d_curved", (45, 52), 190, 0.6, 10, 360, FAN),
    "arc_few_wide_bins": ("fan2d_curved", (26, 26), 4, 40.0, 9, 360, dict(sid=30.0, sdd=60.0)),
    "arc_tiny": ("fan2d_curved", (2, 3), 9, 0.4, 8, 220, FAN),
}


@pytest.fixture(scope="module")
def ph():
    gc.device()
    import paper_1904_13342_amd as ph
    return ph


def _setup(ph, name):
    kind, shape, nu, du, views, turn, src = CASES[name]
    spec = synth.config("par2d_64").with_(kind=kind, vol_shape=shape, vol_spacing=(1.0, 1.0), det_shape=(nu,),
                                          det_spacing=(du,), n_proj=views, angular_range=turn * math.pi / 180, **src)
    g = ph.from_spec(spec)
    fan = kind != "par2d"
    return spec, g, ph.ray_vectors_2d(g), fan


@pytest.mark.parametrize("name", list(CASES))
def test_backproject_adjoint_2d_edges(ph, ora, name):
    import numpy as np
    spec, g, rv, fan = _setup(ph, name)
    rng = np.random.default_rng(5)
    f = as_f32(rng.standard_normal((3,) + spec.vol_shape))
    bT = ph.backproject_adjoint_fan2d if fan else ph.backproject_adjoint_par2d
    out = bT(g, rv, to_dev(f))
    say(f"[B^T 2D] {name}")
    check(to_np(out), np.stack([ora.backproject_adjoint(spec, v) for v in f]), name)
    assert (bT(g, rv, to_dev(f)) == out).all()   # the same bits on every run


@pytest.mark.parametrize("name", list(CASES))
def test_backproject_adjoint_2d_many_items(ph, ora, name):
    """Enough items that a view's workgroup takes whole runs of pixels
    (images up to 128^2 do at any number), and an image large enough that few
    items go by strips."""
    import numpy as np
    spec, g, rv, fan = _setup(ph, name)
    f = as_f32(np.random.default_rng(7).uniform(0.5, 1.5, (2,) + spec.vol_shape))
    bT = ph.backproject_adjoint_fan2d if fan else ph.backproject_adjoint_par2d
    many = -(-256 // spec.n_proj)
    out = bT(g, rv, to_dev(f).repeat(many, 1, 1))
    say(f"[B^T 2D, {2 * many} items] {name}")
    check(to_np(out[:2]), np.stack([ora.backproject_adjoint(spec, v) for v in f]), name)
    assert (out.view((many, 2) + tuple(out.shape[1:])) == out[:2]).all()


@pytest.mark.parametrize("name", list(CASES))
def test_backproject_adjoint_2d_item_pairs(ph, ora, name):
    """An odd number of items, enough that runs take them two at a time."""
    import numpy as np
    import torch
    spec, g, rv, fan = _setup(ph, name)
    f = as_f32(np.random.default_rng(9).uniform(0.5, 1.5, (3,) + spec.vol_shape))
    bT = ph.backproject_adjoint_fan2d if fan else ph.backproject_adjoint_par2d
    pairs = -(-512 // spec.n_proj) + 1
    x = torch.cat([to_dev(f[:2]).repeat(pairs, 1, 1), to_dev(f[2:])])
    out = bT(g, rv, x)
    say(f"[B^T 2D, {2 * pairs + 1} items] {name}")
    check(to_np(out[[0, 1, -1]]), np.stack([ora.backproject_adjoint(spec, v) for v in f]), name)
    assert (out[:-1].view((pairs, 2) + tuple(out.shape[1:])) == out[:2]).all()
    assert (bT(g, rv, x) == out).all()
    # half storage: the sums are FP32, so pairs and single items differ by one rounding at most
    half, one = bT(g, rv, x.half())[:1].float(), bT(g, rv, x[:1].half()).float()
    assert float((half - one).abs().max()) <= 2.0 ** -10 * float(one.abs().max())


@pytest.mark.parametrize("kind,du", [("par2d", 0.6), ("par2d", 1.0), ("par2d", 1.9), ("par2d", 2.5), ("par2d", 3.5),
                                     ("fan2d", 1.1), ("fan2d_curved", 1.9)])
def test_backproject_adjoint_2d_strips_and_runs(ph, ora, kind, du):
    """A 140 x 150 image, a few views (strips) and 260 (runs), for bins of a
    fraction of a pixel to several."""
    import numpy as np
    src = dict(sid=400.0, sdd=640.0) if kind != "par2d" else {}
    fan = kind != "par2d"
    for views in (12, 260):
        spec = synth.config("par2d_64").with_(kind=kind, vol_shape=(140, 150), vol_spacing=(1.0, 1.0),
                                              det_shape=(int(330 / du),), det_spacing=(du,), n_proj=views,
                                              angular_range=2 * math.pi, **src)
        g = ph.from_spec(spec)
        f = as_f32(np.random.default_rng(11).uniform(0.5, 1.5, spec.vol_shape))
        bT = ph.backproject_adjoint_fan2d if fan else ph.backproject_adjoint_par2d
        say(f"[B^T 2D] {kind} bins of {du}, {views} views")
        check(to_np(bT(g, ph.ray_vectors_2d(g), to_dev(f))), ora.backproject_adjoint(spec, f), "B^T")


@pytest.mark.parametrize("name", list(CASES))
def test_project_adjoint_2d_edges(ph, ora, name):
    import numpy as np
    spec, g, rv, fan = _setup(ph, name)
    rng = np.random.default_rng(6)
    p = as_f32(rng.standard_normal((3, spec.n_proj) + spec.det_shape))
    aT = ph.project_adjoint_fan2d if fan else ph.project_adjoint_par2d
    out = aT(g, rv, to_dev(p))
    say(f"[A^T 2D] {name}")
    check(to_np(out), np.stack([ora.project_adjoint(spec, v) for v in p]), name, tol=TOL_AT)
    assert (aT(g, rv, to_dev(p)) == out).all()


@pytest.mark.parametrize("items", [1, 2, 4, 5, 8, 9])
@pytest.mark.parametrize("name", ["par_63", "par_127_fine", "arc_190"])
def test_project_adjoint_2d_item_groups(ph, ora, name, items):
    """Groups of up to eight items with the last one part empty."""
    import numpy as np
    spec, g, rv, fan = _setup(ph, name)
    p = as_f32(np.random.default_rng(13).standard_normal((items, spec.n_proj) + spec.det_shape))
    aT = ph.project_adjoint_fan2d if fan else ph.project_adjoint_par2d
    out = aT(g, rv, to_dev(p))
    say(f"[A^T 2D, {items} items] {name}")
    check(to_np(out), np.stack([ora.project_adjoint(spec, v) for v in p]), name, tol=TOL_AT)


@pytest.mark.parametrize("items", [1, 2, 3, 4, 5, 9])
@pytest.mark.parametrize("kind,du,step", [("par2d", 0.7, 0.0), ("par2d", 0.31, 0.0), ("par2d", 2.2, 0.2),
                                          ("fan2d", 1.1, 0.0), ("fan2d_curved", 0.6, 1.4)])
def test_project_adjoint_2d_tiles_of_eight(ph, ora, kind, du, step, items):
    """Images with enough tiles that the waves hold 8 x 8 pixels, items alone and
    in groups of two, four and eight (the smaller images above have tiles of
    4 x 4); footprints of one, two and more passes of rays."""
    import numpy as np
    src = dict(sid=160.0, sdd=256.0) if kind != "par2d" else {}
    nu = int(135 * (1.7 if src else 1.0) / du)
    spec = synth.config("par2d_64").with_(kind=kind, vol_shape=(90, 101), vol_spacing=(1.0, 1.0), det_shape=(nu,),
                                          det_spacing=(du,), n_proj=7, angular_range=2 * math.pi, step_mm=step, **src)
    g = ph.from_spec(spec)
    p = as_f32(np.random.default_rng(17).standard_normal((items, 7, nu)))
    aT = ph.project_adjoint_fan2d if src else ph.project_adjoint_par2d
    say(f"[A^T 2D, {items} items] {kind} bins of {du}, step {step}")
    out = to_np(aT(g, ph.ray_vectors_2d(g), to_dev(p)))
    for n in {0, items // 2, items - 1}:
        check(out[n], ora.project_adjoint(spec, p[n]), f"item {n}", tol=TOL_AT)


@pytest.mark.parametrize("shape,items,views", [((3, 5), 1, 4), ((64, 61), 2, 13), ((88, 64), 1, 35), ((90, 96), 1, 35)])
@pytest.mark.parametrize("du", [0.2, 1.0, 4.0])
def test_project_adjoint_2d_tiles_of_four(ph, ora, shape, items, views, du):
    """Small images, up to where tiles of 8 x 8 fill half of the GPU and one
    beyond; views in numbers that are no multiple of the four of a wave."""
    import numpy as np
    nu = int(1.45 * max(shape) / du) + 2
    spec = synth.config("par2d_64").with_(vol_shape=shape, vol_spacing=(1.0, 1.0), det_shape=(nu,), det_spacing=(du,),
                                          n_proj=views, angular_range=math.pi)
    g = ph.from_spec(spec)
    p = as_f32(np.random.default_rng(18).standard_normal((items, views, nu)))
    say(f"[A^T 2D] {shape} x {items}, bins of {du}")
    out = to_np(ph.project_adjoint_par2d(g, ph.ray_vectors_2d(g), to_dev(p)))
    check(out, np.stack([ora.project_adjoint(spec, v) for v in p]), "A^T", tol=TOL_AT)


@pytest.mark.parametrize("n", [64, 120])
def test_project_adjoint_2d_not_a_number(ph, n):
    """A ray that is not a number spoils the pixels whose support it crosses, and
    those it misses by a hundredth of a step at most (the clip's tolerance), in
    its own item alone."""
    import numpy as np
    import torch
    views, nu, items = 90, 3 * n // 2, 160
    g = ph.geom2d((n, n), (1.0, 1.0), nu, 1.0, views, math.pi)
    rv = ph.ray_vectors_2d(g)
    p = torch.ones((items, views, nu), device=gc.device())
    at = [((7 * i) % views, (13 * i + 5) % nu) for i in range(items)]
    for i, (k, j) in enumerate(at):
        p[i, k, j] = float("nan")
    bad = torch.isnan(ph.project_adjoint_par2d(g, rv, p)).cpu().numpy()
    ix = np.arange(n, dtype=np.float64)
    step, total = 0.5, 0
    for i, (k, j) in enumerate(at):
        c = rv[k].astype(np.float64) / np.linalg.norm(rv[k].astype(np.float64))
        u = j - 0.5 * (nu - 1)
        X0, Y0 = -u * c[1] + 0.5 * (n - 1), u * c[0] + 0.5 * (n - 1)
        eX, eY = step * c[0], step * c[1]
        # steps at which the ray enters and leaves a pixel's support, per axis
        with np.errstate(divide="ignore", invalid="ignore"):
            tx = np.sort(np.stack([(ix - 1 - X0) / eX, (ix + 1 - X0) / eX]), axis=0)
            ty = np.sort(np.stack([(ix - 1 - Y0) / eY, (ix + 1 - Y0) / eY]), axis=0)
        gap = np.maximum(tx[0][None, :], ty[0][:, None]) - np.minimum(tx[1][None, :], ty[1][:, None])
        if min(abs(eX), abs(eY)) < 1e-6:
            continue
        assert not bad[i][gap > 0.0105].any(), (i, k, j)
        assert bad[i][gap < -1.0].all(), (i, k, j)   # a whole step inside
        total += bad[i].sum()
    assert total > 0
