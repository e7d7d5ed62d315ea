"""LP anti-aliasing of long edges (GPU): flat areas wider than the end search
(8 rows, 8 columns), so that searches run past a tile's staged window, over
the seam of the angle and to the first and last column.  Both forms of the
kernel (layouts below and from 131,072 texels), every texel against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ECC, CPD = [0.0, 10.0, 20.0, 30.0, 60.0], [40.0, 10.0, 6.0, 5.0, 4.0]


def _buffer(kind, layout):
    """RGBA per texel from its column and its angle in turns."""
    rows, off = np.asarray(layout.n_rows, np.int64), np.asarray(layout.col_off, np.int64)
    col = np.repeat(np.arange(layout.n_cols), rows)
    row = np.arange(layout.n_texels) - off[col]
    turns = (row + 0.5) / rows[col]
    lo, hi = np.float32([0.1, 0.2, 0.05, 1.0]), np.float32([0.9, 0.7, 0.8, 0.5])
    if kind == "ring":               # an edge along the angle, right round the seam
        on = col >= layout.n_cols // 2
    elif kind == "half":             # two edges along the radius, one on the seam
        on = turns < 0.5
    elif kind == "wedge":            # an edge along the radius that meets one along the angle
        on = (turns > 0.97) | (turns < 0.04) | (col < 3)
    elif kind == "spiral":           # an edge that steps by a row every few columns
        on = ((turns + col / 150.0) % 0.25) < 0.125
    else:                            # blocks of 11 columns by 13 rows
        rng = np.random.default_rng(5)
        value = rng.random((layout.n_cols // 11 + 1, int(rows.max()) // 13 + 1, 4)).astype(np.float32)
        return np.ascontiguousarray(value[col // 11, row // 13])
    return np.ascontiguousarray(np.where(on[:, None], hi, lo))


@pytest.mark.parametrize("e_max", [0.6, 3.0, 8.0, 60.0])
@pytest.mark.parametrize("kind", ["ring", "half", "wedge", "spiral", "blocks"])
def test_long_edges_match_the_oracle(O, e_max, kind):
    import torch
    from paper_2503_23410_amd import vafr as V
    L = V.Layout.vafr(V.display(640, 360), ECC, CPD, e_max)
    ref = O.Layout(O.Acuity(ECC, CPD), e_max)
    assert L.n_texels == ref.n_texels
    lp = _buffer(kind, ref)
    out = torch.full((L.n_texels, 4), float("nan"), device="cuda")
    V.vafr_fxaa_lp(L, torch.from_numpy(lp).cuda(), out)
    torch.cuda.synchronize()
    want = O.fxaa_lp(ref, lp)
    assert np.abs(out.cpu().numpy() - want).max() <= 2e-3
    assert np.abs(want - lp).max() > 0.03      # edges were blended


# layouts just below and just above the line between the two forms
@pytest.mark.parametrize("e_max,direct", [(4.6, True), (4.7, False)])
def test_both_forms_give_one_image(O, e_max, direct):
    import torch
    from paper_2503_23410_amd import inputs as I
    from paper_2503_23410_amd import vafr as V
    L = V.Layout.vafr(V.display(640, 360), ECC, CPD, e_max)
    assert (L.n_texels < 131072) == direct, L.n_texels
    ref = O.Layout(O.Acuity(ECC, CPD), e_max)
    lp = I.random_lp(L.n_texels, seed=3)
    out = torch.empty((L.n_texels, 4), device="cuda")
    V.vafr_fxaa_lp(L, torch.from_numpy(lp).cuda(), out)
    torch.cuda.synchronize()
    assert np.abs(out.cpu().numpy() - O.fxaa_lp(ref, lp)).max() <= 2e-3
