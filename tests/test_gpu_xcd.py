"""Dealing of traversal work to the XCDs in batches (GPU): every ray is traced
exactly once whatever the workgroup size and the number of workgroups, in the
first frame and in the second, which follows the order that the first one's
durations planned."""
import pytest

from paper_2503_23410_amd import inputs as I

pytestmark = pytest.mark.gpu


# 8 x 8 pixel tiles, one, two or four per workgroup of 64, 128 or 256 rays; a
# chunk is 16 tiles, one round of chunks over 8 XCDs 128: fewer workgroups than
# XCDs, a workgroup less and more than a round, ragged rests.
@pytest.mark.parametrize("block", [64, 128, 256])
@pytest.mark.parametrize("use_graph", [False, True])
def test_batch_traces_every_tile_once(block, use_graph):
    import torch
    from paper_2503_23410_amd import vafr as V
    scene, sh, cam = V.Scene(*I.soup_scene(64, seed=4)), V.shading(), V.camera(I.soup_camera())
    H = 5
    for tiles in (1, 2, 5, 13, 16, 29, 31, 32, 33, 61, 64, 124, 126, 127, 128, 129, 130, 132, 160, 254, 256, 1000, 1023,
                  1024, 1040, 2047):
        W = 8 * tiles
        one, one_id = torch.empty((W * H, 4), device="cuda"), torch.empty(W * H, device="cuda", dtype=torch.int32)
        V.full_shade(scene, cam, V.display(W, H), sh, one, one_id)
        img, hid = torch.empty_like(one), torch.empty_like(one_id)
        b = V.Batch(1, trace_block=block, use_graph=use_graph)
        view = V.view(V.VAFR_VIEW_FULL, scene, cam, V.gaze(0.0, 0.0), sh, disp=V.display(W, H), hit_id=hid, img_rgba=img)
        for frame in range(3):
            img.fill_(float("nan"))
            hid.fill_(-7)
            b.run([view])
            torch.cuda.synchronize()
            assert torch.equal(hid, one_id) and torch.equal(img, one), (tiles, frame)
        b.close()


# several views in one launch, cut across workgroups, chunks and XCDs
@pytest.mark.parametrize("block", [64, 128, 256])
def test_batch_of_ragged_views(block):
    import torch
    from paper_2503_23410_amd import vafr as V
    scene, sh, cam = V.Scene(*I.soup_scene(64, seed=4)), V.shading(), V.camera(I.soup_camera())
    sizes = [(8, 3), (1000, 9), (17, 40), (8 * 127, 8), (8 * 129, 8), (3, 3), (515, 77)]
    one = [torch.empty((w * h, 4), device="cuda") for w, h in sizes]
    img = [torch.empty_like(x) for x in one]
    for (w, h), x in zip(sizes, one):
        V.full_shade(scene, cam, V.display(w, h), sh, x)
    views = [V.view(V.VAFR_VIEW_FULL, scene, cam, V.gaze(0.0, 0.0), sh, disp=V.display(w, h), img_rgba=x)
             for (w, h), x in zip(sizes, img)]
    b = V.Batch(len(sizes), trace_block=block)
    for frame in range(3):
        for x in img:
            x.fill_(float("nan"))
        b.run(views)
        torch.cuda.synchronize()
        for k in range(len(sizes)):
            assert torch.equal(img[k], one[k]), (k, frame)
    b.close()
