"""The node format that the traversal relies on (CPU): the fast box test,
formed here operation by operation in FP32 on nodes brought into the device's
format, never meets an empty slot and always meets a child whose triangles'
box the exact ray meets -- for origins up to the scene's limit, directions from
the smallest to the largest that the form takes and along the axes."""
import numpy as np
import pytest

from paper_2503_23410_amd import inputs as I

F = np.float32
EMPTY = np.iinfo(np.int32).min
TINY = F(2.0 ** -57)


def fma(a, b, c):
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(F)


def _scenes():
    v, f = I.soup_scene(300, seed=9)
    yield "soup", v, f
    v, f = I.terrain_scene(32, 16, 4, seed=5)
    yield "terrain", v, f
    yield "small", v * F(1e-3), f
    yield "large", v * F(1e6), f
    yield "three", *I.soup_scene(9, seed=1)


def _child_boxes(nodes, order, verts, tris):
    """Exact box of the triangles under each child, (n, 4, 2, 3)."""
    refs = nodes[:, 12:16].view(np.int32)
    tv = verts[tris[order]].astype(np.float64)
    box = np.full((len(nodes), 4, 2, 3), np.nan)
    for n in range(len(nodes) - 1, -1, -1):      # children follow their parent
        for c in range(4):
            r = refs[n, c]
            if r == EMPTY:
                continue
            if r < 0:
                first, cnt = (~r) >> 3, ((~r) & 7) + 1
                p = tv[first:first + cnt].reshape(-1, 3)
                box[n, c] = p.min(0), p.max(0)
            else:
                box[n, c] = np.nanmin(box[r, :, 0], 0), np.nanmax(box[r, :, 1], 0)
    return refs, box


def _fast(nodes, refs, o, d):
    """The fast box test: whether the ray meets each child of each node."""
    codes = np.ascontiguousarray(nodes[:, 4:12]).view(np.uint32)[:, :6].copy()
    empty = refs == EMPTY
    for c in range(4):       # the device's format
        b = np.uint32(255 << (8 * c))
        codes[empty[:, c], 0::2] |= b
        codes[empty[:, c], 1::2] &= ~b
    near, far = [], []
    for a in range(3):
        scale = nodes[:, (10, 11, 3)[a]] * F(2.0 ** 49)
        org = nodes[:, a] * F(2.0 ** -100)
        da = np.copysign(TINY, d[a]) if abs(d[a]) < TINY else d[a]
        inv = F(1.0) / da
        oi = F(F(o[a] * inv) * F(2.0 ** -100))
        base = fma(org, np.full_like(org, inv), np.full_like(org, -oi))
        lo, hi = codes[:, 2 * a], codes[:, 2 * a + 1]
        if inv < 0:
            lo, hi = hi, lo
        planes = []
        for w in (lo, hi):
            q = np.stack([(w & np.uint32(0xff << (8 * c))) if c < 3 else w >> 24 for c in range(4)], 1)
            t = np.stack([scale * inv * F(2.0 ** (-8 * (c % 3))) for c in range(4)], 1).astype(F)
            planes.append(fma(np.ascontiguousarray(q, np.uint32).view(F), t, base[:, None]))
        near.append(planes[0])
        far.append(planes[1])
    n, f = np.max(near, 0), np.min(far, 0)
    return ~(np.signbit(f - n) | np.signbit(f))


def _exact(box, o, d):
    """Whether the exact ray meets each child's box at t >= 0 (FP64; planes of
    axes along which it does not move are tested by position)."""
    o, d = o.astype(np.float64), d.astype(np.float64)
    t0, t1 = np.zeros(box.shape[:2]), np.full(box.shape[:2], np.inf)
    for a in range(3):
        lo, hi = box[:, :, 0, a], box[:, :, 1, a]
        if d[a] == 0.0:
            t1 = np.where((o[a] >= lo) & (o[a] <= hi), t1, -np.inf)
            continue
        x, y = (lo - o[a]) / d[a], (hi - o[a]) / d[a]
        t0, t1 = np.maximum(t0, np.minimum(x, y)), np.minimum(t1, np.maximum(x, y))
    return t0 <= t1


@pytest.mark.parametrize("name,verts,tris", list(_scenes()), ids=[s[0] for s in _scenes()])
def test_fast_form_keeps_boxes_and_drops_empty_slots(name, verts, tris):
    from paper_2503_23410_amd import vafr as V
    verts = np.ascontiguousarray(verts, F)
    nodes, order = V.Scene(verts, tris).export()
    refs, box = _child_boxes(nodes, order, verts, tris)
    empty = refs == EMPTY
    ext = np.abs(verts[np.unique(tris)]).max()
    pad = F(2e-5) * (F(1.0) + ext)
    span = 255.0 * nodes[:, [10, 11, 3]].astype(np.float64)
    assert (span >= 2.0 * pad * (1 - 1e-6)).all()    # an empty slot is inside out by at least this
    codes = np.ascontiguousarray(nodes[:, 4:12]).view(np.uint32)[:, :6]
    for c in range(4):
        assert ((codes[empty[:, c]] >> np.uint32(8 * c)) & 255 == 0).all()
    limit = max(0.0, min(float(pad) * 524288.0 - float(ext), 1e7))
    rng = np.random.default_rng(11)
    with np.errstate(all="ignore"):
        for k in range(120):
            # origins inside the scene, on its surface and at the limit
            if k % 3 == 2:
                o = rng.uniform(-1, 1, 3) * limit
                o[rng.integers(3)] = limit * rng.choice([-1, 1])
                target = box[rng.integers(len(box)), 0].mean(0)
                d = target - o
            else:
                o = verts[tris[rng.integers(len(tris))]].mean(0) + rng.normal(size=3) * (ext * 0.3 if k % 3 else 1e-3)
                d = rng.normal(size=3)
            if k % 4 == 1:       # one component zero, two of them (or far below the form's smallest)
                d[rng.integers(3)] = 0.0 * rng.choice([-1.0, 1.0])
            if k % 8 == 3:
                a = rng.integers(3)
                d = np.where(np.arange(3) == a, np.sign(d[a]) or 1.0, rng.choice([-0.0, 0.0, 1e-30, -1e-20], 3))
            d = d / np.abs(d).max()
            o = o.astype(F)
            d = (d * 2.0 ** rng.choice([-9.0, 0.0, 0.0, 19.0])).astype(F)
            assert np.abs(o).max() <= limit * (1 + 1e-6) and 2.0 ** -10 <= np.abs(d).max() <= 2.0 ** 20
            met = _fast(nodes, refs, o, d)
            assert not met[empty].any(), (k, o, d)
            need = _exact(np.where(np.isnan(box), 0.0, box), o, d) & ~empty
            assert met[need].all(), (k, o, d, int((need & ~met).sum()))
