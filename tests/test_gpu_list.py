"""The reprojection's list of uncovered texels (GPU): lists of at most a fifth
of the texels, whose Lambert-shaded rays four lanes share, and longer ones.
Every uncovered texel must equal the directly shaded one, bit for bit."""
import numpy as np
import pytest

from paper_2503_23410_amd import inputs as I

pytestmark = pytest.mark.gpu


# How far the right eye stands from the left one sets the length of the list;
# the last column says on which side of a fifth it falls.
@pytest.mark.parametrize("scene_name,e_max,apart,short", [
    ("terrain", 60.0, 0.064, True), ("terrain", 60.0, 0.3, True), ("terrain", 12.0, 0.064, True),
    ("terrain", 60.0, 3.0, False), ("soup", 60.0, 0.02, False), ("soup", 60.0, 0.5, False),
])
@pytest.mark.parametrize("mode", ["lambert", "unshadowed", "path"])
def test_uncovered_texels_equal_the_shaded_ones(scene_name, e_max, apart, short, mode):
    import torch
    from paper_2503_23410_amd import vafr as V
    soup = scene_name == "soup"
    scene = V.Scene(*(I.soup_scene(40, seed=8) if soup else I.terrain_scene(64, 32, 9, seed=5)))
    cam = np.array(I.soup_camera() if soup else I.terrain_camera(), np.float32)
    right = cam.copy()
    right[:3] += np.float32(apart) * cam[3:6]
    L = V.Layout.vafr(V.display(640, 360), [0.0, 10.0, 20.0, 30.0, 60.0], [40.0, 10.0, 6.0, 5.0, 4.0], e_max)
    n = L.n_texels
    gaze = V.gaze(300.0, 170.0)
    sh = V.shading(mode=V.VAFR_SHADE_PATH, bounces=1, seed=3) if mode == "path" else V.shading(shadow=mode == "lambert")
    lp = [torch.full((n, 4), float("nan"), device="cuda") for _ in range(3)]
    ids = [torch.full((n,), -7, device="cuda", dtype=torch.int32) for _ in range(3)]
    ws = torch.empty(V.rep_workspace_bytes(L), device="cuda", dtype=torch.uint8)
    V.vafr_shade_lp_rep(scene, V.camera(cam), V.camera(right), gaze, sh, L, lp[0], lp[1], ws, ids[0], ids[1])
    V.vafr_shade_lp(scene, V.camera(right), gaze, sh, L, lp[2], ids[2])
    torch.cuda.synchronize()
    # the workspace holds n hit points of 16 bytes, then a key per texel, all
    # ones where the left eye's grid covers nothing
    holes = ws[16 * n:24 * n].view(torch.int64) == -1
    listed = int(holes.sum())
    print(f"{listed} of {n} texels listed")
    assert listed > 0 and (5 * listed <= n) == short
    assert torch.equal(ids[1][holes], ids[2][holes])
    assert torch.equal(lp[1][holes], lp[2][holes])
    assert not torch.isnan(lp[1]).any()
