"""Traversal launches (GPU): every ray is traced exactly once whatever the
number of workgroups, and both forms of the slab test agree with the oracle
at the ends of the fast form's range."""
import numpy as np
import pytest

from paper_2503_23410_amd import inputs as I

pytestmark = pytest.mark.gpu


# 8 x 8 pixel tiles, two per 128-ray workgroup, chunks of 8 workgroups dealt
# to 8 XCDs: fewer workgroups than XCDs, one chunk per XCD less one, exactly
# one, one more, and several chunks with a ragged rest.
# (Those are the workgroups of a batch; a per-view launch has one tile per
# 64-ray workgroup and chunks of 16.  Batches: test_gpu_xcd.py.)
@pytest.mark.parametrize("tiles", [1, 2, 13, 16, 17, 126, 128, 130, 254, 1000, 1023, 1024, 1040, 2047])
def test_full_shade_traces_every_tile_once(O, tiles):
    import torch
    from paper_2503_23410_amd import vafr as V
    v, f = I.soup_scene(64, seed=4)
    W, H = 8 * tiles, 5
    scene, cam = V.Scene(v, f), I.soup_camera()
    img = torch.full((W * H, 4), float("nan"), device="cuda")
    hid = torch.full((W * H,), -7, device="cuda", dtype=torch.int32)
    V.full_shade(scene, V.camera(cam), V.display(W, H), V.shading(), img, hid)
    torch.cuda.synchronize()
    osc = O.Scene(v, f)
    rgba, ids, flags = O.shade_full_pixels(osc, np.arange(W * H), W, H, I.FOV, cam, O.shading_params())
    ok = flags == 0
    assert np.array_equal(hid.cpu().numpy()[ok], ids[ok])
    assert np.abs(img.cpu().numpy() - rgba)[ok].max() <= 2e-3


# The fast slab form takes directions whose largest component lies in
# [2^-10, 2^20] and raises components below 2^-57; the general form takes the
# rest.  The camera's basis scaled by a power of two scales every direction by
# it (and every hit distance by its inverse), so the oracle's hits follow.
@pytest.mark.parametrize("shift", [-60, -12, -10, -8, 0, 17, 19, 21])
@pytest.mark.parametrize("scene_name", ["soup", "terrain"])
def test_direction_scales(O, shift, scene_name):
    import torch
    from paper_2503_23410_amd import vafr as V
    v, f = I.soup_scene(300, seed=9) if scene_name == "soup" else I.terrain_scene(48, 24, 9, seed=5)
    cam = np.array(I.soup_camera() if scene_name == "soup" else I.terrain_camera(), np.float32)
    cam[3:] *= np.float32(2.0 ** shift)
    W, H = 161, 95
    scene = V.Scene(v, f)
    img = torch.empty((W * H, 4), device="cuda")
    hid = torch.empty(W * H, device="cuda", dtype=torch.int32)
    V.full_shade(scene, V.camera(cam), V.display(W, H), V.shading(), img, hid)
    torch.cuda.synchronize()
    osc = O.Scene(v, f)
    rgba, ids, flags = O.shade_full_pixels(osc, np.arange(W * H), W, H, I.FOV, cam, O.shading_params())
    ok = flags == 0
    assert ok.mean() > 0.99 and (ids >= 0).mean() > 0.05
    assert np.array_equal(hid.cpu().numpy()[ok], ids[ok])
    assert np.abs(img.cpu().numpy() - rgba)[ok].max() <= 2e-3


# Rays along the axes: odd displays put a row and a column of pixel centres
# exactly on the camera's axes, so primary rays there have one or two zero
# components, and the light's rays have two.
@pytest.mark.parametrize("light", [(0.0, 1.0, 0.0), (0.0, 0.0, -1.0), (-1.0, 0.0, 0.0), (1e-20, 1.0, -1e-25)])
def test_axis_parallel_rays(O, light):
    import torch
    from paper_2503_23410_amd import vafr as V
    v, f = I.soup_scene(500, seed=3)
    cam = I.soup_camera()
    W, H = 129, 77
    scene = V.Scene(v, f)
    img = torch.empty((W * H, 4), device="cuda")
    hid = torch.empty(W * H, device="cuda", dtype=torch.int32)
    V.full_shade(scene, V.camera(cam), V.display(W, H), V.shading(light_dir=light), img, hid)
    torch.cuda.synchronize()
    osc = O.Scene(v, f)
    rgba, ids, flags = O.shade_full_pixels(osc, np.arange(W * H), W, H, I.FOV, cam,
                                           O.shading_params(light_dir=light))
    ok = flags == 0
    assert ok.mean() > 0.99
    assert np.array_equal(hid.cpu().numpy()[ok], ids[ok])
    assert np.abs(img.cpu().numpy() - rgba)[ok].max() <= 2e-3


# The reprojection's list of uncovered texels: a left eye that looks away from
# the scene hits nothing, so nothing is warped, every texel of the right eye is
# listed and must equal the directly shaded one.  Short lists (four lanes per Lambert-shaded ray, whose
# way is cut into segments), long ones, and path-traced ones; the far eyes see
# the scene's box from outside, from afar and not at all.
@pytest.mark.parametrize("e_max", [0.1, 3.0, 60.0])
@pytest.mark.parametrize("mode", ["lambert", "unshadowed", "path"])
@pytest.mark.parametrize("eye", [(0.1, 0.2, 0.3), (0.0, 0.0, 40.0), (3.0e4, 10.0, 2.0e4)])
def test_listed_texels_equal_the_shaded_ones(e_max, mode, eye):
    import torch
    from paper_2503_23410_amd import vafr as V
    scene = V.Scene(*I.soup_scene(2000, seed=8))
    L = V.Layout.vafr(V.display(640, 360), [0.0, 10.0, 20.0, 30.0, 60.0], [40.0, 10.0, 6.0, 5.0, 4.0], e_max)
    left = np.array([0, 0, -3, -1, 0, 0, 0, 1, 0, 0, 0, -1], np.float32)
    right = np.array([*eye, -1, 0, 0, 0, 1, 0, 0, 0, -1], np.float32)
    gaze = V.gaze(300.0, 170.0)
    sh = V.shading(mode=V.VAFR_SHADE_PATH, bounces=1, seed=3) if mode == "path" else V.shading(shadow=mode == "lambert")
    lp = [torch.full((L.n_texels, 4), float("nan"), device="cuda") for _ in range(3)]
    ids = [torch.full((L.n_texels,), -7, device="cuda", dtype=torch.int32) for _ in range(3)]
    ws = torch.empty(V.rep_workspace_bytes(L), device="cuda", dtype=torch.uint8)
    V.vafr_shade_lp_rep(scene, V.camera(left), V.camera(right), gaze, sh, L, lp[0], lp[1], ws, ids[0], ids[1])
    V.vafr_shade_lp(scene, V.camera(right), gaze, sh, L, lp[2], ids[2])
    torch.cuda.synchronize()
    assert torch.equal(ids[1], ids[2])
    assert torch.equal(lp[1], lp[2])
