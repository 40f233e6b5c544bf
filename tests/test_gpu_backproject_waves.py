"""The 3D back-projector's wave kernel (small volumes and general matrices)
against the FP64 oracle at the edges of its tiles, on detectors that some
voxels miss, in every storage type, and against the brick kernel where the
dispatch changes from one to the other."""
import math

import numpy as np
import pytest
import torch

import gpu_common as gc
import synth
from gpu_common import as_f32, check, say, to_dev, to_np

pytestmark = pytest.mark.gpu

BASE = synth.config("cone3d_crop32").with_(vol_spacing=(1.0, 1.0, 1.0), det_spacing=(1.4, 1.3), sid=300.0, sdd=500.0,
                                           angular_range=200 * math.pi / 180)
# vol shape, detector, views
CASES = {
    "one_voxel": ((1, 1, 1), (5, 7), 3),
    "tile_edges": ((5, 9, 8), (21, 25), 17),
    "tile_plus_one": ((33, 17, 25), (60, 50), 64),
    "misses_rows": ((40, 16, 24), (9, 41), 12),
    "misses_columns": ((12, 40, 44), (31, 12), 12),
    "one_row_detector": ((4, 24, 24), (1, 40), 20),
    "one_column_detector": ((4, 24, 24), (11, 1), 20),
}


@pytest.fixture(scope="module")
def ph():
    gc.device()
    import paper_1904_13342_amd as ph
    return ph


@pytest.mark.parametrize("orbit", ["circle", "perturbed"])
@pytest.mark.parametrize("name", list(CASES))
def test_backproject_waves(ph, ora, name, orbit):
    vol, det, views = CASES[name]
    spec = BASE.with_(vol_shape=vol, det_shape=det, n_proj=views)
    g = ph.from_spec(spec)
    if orbit == "circle":
        mats, kw = ph.projection_matrices_3d(g), {}
    else:
        mats = synth.pose_matrices(spec, synth.perturbed_poses(spec, 4)).astype(np.float32)
        kw = dict(mats=mats.astype(np.float64))
    p = as_f32(np.random.default_rng(2).uniform(0.5, 1.5, (2, views) + det))
    ref = np.stack([ora.backproject(spec, v, **kw) for v in p])
    say(f"[B waves] {name} {orbit}")
    check(to_np(ph.backproject_cone3d(g, mats, to_dev(p))), ref, "f32")
    for dt, key, tol in ((torch.float16, "f16", 2e-3), (torch.bfloat16, "bf16", 1e-2)):
        q = to_dev(p).to(dt)
        refq = np.stack([ora.backproject(spec, v, **kw) for v in q.double().cpu().numpy()])
        check(to_np(ph.backproject_cone3d(g, mats, q)), refq, key, tol=tol, elem=gc.ELEM_TOL_HALF[key])


def test_waves_and_bricks_agree(ph):
    """One item is 256 bricks (waves), three are 768 (bricks)."""
    spec = BASE.with_(vol_shape=(20, 250, 256), det_shape=(60, 400), n_proj=30)
    g = ph.from_spec(spec)
    mats = ph.projection_matrices_3d(g)
    gen = torch.Generator(device=gc.device()).manual_seed(5)
    p = torch.rand((3, 30, 60, 400), device=gc.device(), generator=gen)
    whole = ph.backproject_cone3d(g, mats, p)
    for b in range(3):
        check(to_np(ph.backproject_cone3d(g, mats, p[b].contiguous())), to_np(whole[b]), f"item {b}")


@pytest.mark.parametrize("det_spacing", [(2.4, 2.3), (0.9, 0.8)])
def test_bricks_by_voxels(ph, ora, det_spacing):
    """Fewer than 512 bricks, but voxels enough that they beat the waves; columns
    of 32 and of 16 voxels."""
    vol, views = (150, 150, 139), 5
    n = int(150 * 1.75 / det_spacing[1])
    spec = BASE.with_(vol_shape=vol, det_shape=(n, n), det_spacing=det_spacing, n_proj=views, sid=700.0, sdd=1100.0)
    g = ph.from_spec(spec)
    p = as_f32(np.random.default_rng(6).uniform(0.5, 1.5, (views, n, n)))
    say(f"[B bricks] {vol}, pixels {det_spacing}")
    check(to_np(ph.backproject_cone3d(g, ph.projection_matrices_3d(g), to_dev(p))), ora.backproject(spec, p), "B")


@pytest.mark.parametrize("views", [9, 24, 25, 60])
def test_backproject_adjoint_shares_of_large_volumes(ph, ora, views):
    """B^T with one, two and three shares of a few hundred bricks."""
    vol = (130, 140, 150)
    spec = BASE.with_(vol_shape=vol, det_shape=(60, 70), det_spacing=(5.0, 5.0), n_proj=views, sid=700.0, sdd=1100.0)
    g = ph.from_spec(spec)
    f = as_f32(np.random.default_rng(7).uniform(0.5, 1.5, vol))
    say(f"[B^T shares] {vol}, {views} views")
    check(to_np(ph.backproject_adjoint_cone3d(g, ph.projection_matrices_3d(g), to_dev(f))),
          ora.backproject_adjoint(spec, f), "B^T")
