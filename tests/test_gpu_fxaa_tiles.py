"""Tiles of the LP anti-aliasing (GPU): layouts whose columns hold one row, a
few rows, just over a tile's 64 rows, and rows that differ sharply between
neighbouring columns, every texel against the oracle."""
import numpy as np
import pytest

from paper_2503_23410_amd import inputs as I

pytestmark = pytest.mark.gpu

ECC, CPD = [0.0, 10.0, 20.0, 30.0, 60.0], [40.0, 10.0, 6.0, 5.0, 4.0]


@pytest.mark.parametrize("e_max", [0.05, 0.6, 3.0, 60.0])
@pytest.mark.parametrize("delta", [([0.0], [1.0]), ([0.0], [1e-3]), ([0.0], [0.04]), ([0.0, 1.0, 1.01], [1.0, 1.0, 0.1])])
def test_every_texel_matches_the_oracle(O, e_max, delta):
    import torch
    from paper_2503_23410_amd import vafr as V
    L = V.Layout.vafr(V.display(640, 360), ECC, CPD, e_max, aniso=delta)
    ref = O.Layout(O.Acuity(ECC, CPD, aniso=delta), e_max)
    assert L.n_texels == ref.n_texels
    lp = I.random_lp(L.n_texels, seed=7)
    lp[::3] = lp[0]     # flat patches: long searches
    out = torch.full((L.n_texels, 4), float("nan"), device="cuda")
    V.vafr_fxaa_lp(L, torch.from_numpy(lp).cuda(), out)
    torch.cuda.synchronize()
    assert np.abs(out.cpu().numpy() - O.fxaa_lp(ref, lp)).max() <= 2e-3
