"""Dispatch order of the traversal launches: every ray is traced exactly once
whatever the number of workgroups (GPU)."""
import numpy as np
import pytest

from paper_2503_23410_amd import inputs as I

pytestmark = pytest.mark.gpu


# 8 x 8 pixel tiles, two per 128-ray workgroup, chunks of 8 workgroups dealt
# to 8 XCDs: fewer workgroups than XCDs, one chunk per XCD less one, exactly
# one, one more, and several chunks with a ragged rest.
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
