"""Timing cases of the VaFR library: the calls a renderer makes per frame.

Each case is a plain dict; `prepare` builds what a program holds before the
frame (resident scene, layout, cameras, buffers, batch handle), `run` makes
the frame's calls once and returns the buffers they wrote.

The kinds of call:
  map      the inverse map of a VaFR LP buffer onto one display
  densemap the inverse map of an LMFR or LaFR buffer
  eye      one eye through the per-view calls: shade the LP buffer (with hit
           ids), then map it to the display
  dense    the same through the LMFR or LaFR calls (the comparison methods)
  full     one eye ray-cast at full resolution (the ground truth)
  frame    a binocular frame through a Batch (graph replay), Lambert + shadow
           rays or path-traced
  mix      one Batch over several independent views of mixed display sizes
  fxaa     anti-aliasing of a shaded LP buffer
  rep      a binocular frame whose right eye is warped from the left one

The seed moves the eye and the gaze, draws the random LP buffers and keys the
path tracer's random numbers.  Terrains are resident assets (one scene serves
every frame and every headset), built once per process.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2503_23410_amd import inputs as I
from paper_2503_23410_amd import vafr as V

# LaFR(2.2) and LMFR(1.8): the buffer scales of the compared methods.
DELTA = {"lmfr": 1.8, "lafr": 2.2}
ECC, CPD, E_MAX = (0.0, 10.0, 20.0, 30.0, 60.0), (40.0, 10.0, 6.0, 5.0, 4.0), 60.0


def listed():
    return [
        # smallest call: a VaFR LP buffer mapped to the test-sized display
        {"name": "map 640x360", "kind": "map", "w": 640, "h": 360},
        # one eye's inverse map at the headline display
        {"name": "map 7680x4320", "kind": "map", "w": 7680, "h": 4320},
        # a log-polar comparison buffer mapped to a ragged 4K-class display
        {"name": "lafr map 3839x2161", "kind": "densemap", "method": "lafr", "w": 3839, "h": 2161},
        # one eye of the small configuration: 4,096-triangle soup
        {"name": "eye soup 640x360", "kind": "eye", "scene": "soup", "size": 4096, "w": 640, "h": 360,
         "acuity": "standard"},
        # one eye, 1.13M triangles, odd display, curve adapted to a 9 cpd panel
        {"name": "eye terrain1m 1921x1083", "kind": "eye", "scene": "terrain", "size": 1024, "w": 1921, "h": 1083,
         "acuity": "cap9"},
        # the headline: binocular 8K frame, 4.52M triangles, one light
        {"name": "frame terrain4m 7680x4320", "kind": "frame", "scene": "terrain", "size": 2048, "w": 7680,
         "h": 4320, "bounces": -1},
        # a served request: binocular 4K, path-traced, 2 bounces
        {"name": "path terrain1m 3840x2160", "kind": "frame", "scene": "terrain", "size": 1024, "w": 3840,
         "h": 2160, "bounces": 2},
        # several headsets' views in one batch (sizes drawn from 720p .. 8K)
        {"name": "mix16 terrain4m", "kind": "mix", "scene": "terrain", "size": 2048, "views": 16, "mixseed": 4},
        # ground truth: full-resolution ray cast of one eye
        {"name": "full terrain1m 2560x1440", "kind": "full", "scene": "terrain", "size": 1024, "w": 2560,
         "h": 1440},
        # comparison method at the headline display
        {"name": "lmfr terrain4m 7680x4320", "kind": "dense", "method": "lmfr", "scene": "terrain", "size": 2048,
         "w": 7680, "h": 4320},
        # anti-aliasing of one shaded LP buffer
        {"name": "fxaa terrain4m", "kind": "fxaa", "scene": "terrain", "size": 2048, "w": 3840, "h": 2160},
        # right eye warped from the left one, then both mapped
        {"name": "rep terrain4m 2560x1440", "kind": "rep", "scene": "terrain", "size": 2048, "w": 2560, "h": 1440},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("map", "densemap", "eye", "eye", "dense", "full", "frame", "frame", "mix", "fxaa", "rep"))
    # the largest ray cast stays below the listed batch of 16 views
    w = _log_uniform(rng, 640, 5120 if kind == "full" else 7680)
    h = max(360, min(4320, int(round(w * rng.choice((9 / 16, 9 / 16, 1.0, 10 / 9)))) + rng.randrange(-3, 4)))
    case = {"kind": kind, "w": w, "h": h}
    if kind in ("densemap", "dense"):
        case["method"] = rng.choice(("lmfr", "lafr"))
    if kind not in ("map", "densemap"):
        # a soup's triangles are as large as the scene: rays visit far more of its tree
        if kind in ("eye", "fxaa") and rng.random() < 0.3:
            case["scene"], case["size"] = "soup", _log_uniform(rng, 64, 4096)
        else:   # size * size / 2 cells of two triangles, and spheres: 17 thousand to 4.5 million triangles
            case["scene"], case["size"] = "terrain", _log_uniform(rng, 128, 2048) // 8 * 8
    if kind == "eye":
        case["acuity"] = rng.choice(("standard", "cap9", "cap18", "aniso"))
    if kind == "frame":
        case["bounces"] = rng.choice((-1, -1, 0, 1, 2, 2))
    if kind == "mix":
        case.pop("w")
        case.pop("h")
        case["views"], case["mixseed"] = rng.randrange(3, 13), rng.randrange(1000)
    return case


# ------------------------------------------------------------------ inputs

@functools.lru_cache(maxsize=3)
def _terrain(size):
    seed = {1024: 2, 2048: 3}.get(size, size)
    return V.Scene(*I.terrain_scene(size, size // 2, size * size // 4096, seed))


def _scene(case, seed):
    """(scene, its vertices, its triangles): the soup's come from the seed."""
    if case["scene"] == "soup":
        v, f = I.soup_scene(case["size"], seed)
        return V.Scene(v, f), v, f
    return _terrain(case["size"]), None, None


def _cameras(case, seed):
    """Left and right eye (12 floats each), the head moved by the seed."""
    rng = np.random.default_rng([seed, 1])
    move = rng.uniform(-0.05, 0.05, 3).astype(np.float32)
    if case["scene"] == "soup":
        pair = [I.soup_camera(), I.soup_camera()]
        pair[0][0] -= 0.5 * I.IPD
        pair[1][0] += 0.5 * I.IPD
    else:
        pair = [c.copy() for c in I.binocular_cameras()]
    for c in pair:
        c[:3] += move
    return pair


def _gaze(w, h, seed, k=0):
    x, y = I.uniform_gaze(1, w, h, seed=seed * 7 + k)[0]
    return float(x), float(y)


def _layout(case, w, h):
    disp = V.display(w, h, I.FOV)
    method = case.get("method")
    if method == "lmfr":
        return V.Layout.lmfr(disp, DELTA["lmfr"])
    if method == "lafr":
        return V.Layout.lafr(disp, DELTA["lafr"])
    acuity = case.get("acuity", "standard")
    if acuity == "cap9":
        return V.Layout.vafr(disp, *V.acuity_capped(9.0))
    if acuity == "cap18":
        return V.Layout.vafr(disp, *V.acuity_capped(18.0))
    if acuity == "aniso":
        return V.Layout.vafr(disp, aniso=((0.0, 30.0), (1.0, 0.5)))
    return V.Layout.vafr(disp)


def _rgba(n):
    return torch.empty((n, 4), device="cuda", dtype=torch.float32)


def _ids(n):
    return torch.empty(n, device="cuda", dtype=torch.int32)


def _random_lp(n, seed):
    return torch.rand((n, 4), generator=torch.Generator("cuda").manual_seed(seed), device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind, "method": case.get("method")}
    if kind == "mix":
        sizes, gazes = I.batch_views(case["views"], seed=case["mixseed"])
        s["scene"], _, _ = _scene(case, seed)
        cam = V.camera(_cameras(case, seed)[0])
        s["layouts"] = [_layout(case, w, h) for w, h in sizes]
        s["lp"] = [_rgba(L.n_texels) for L in s["layouts"]]
        s["img"] = [_rgba(w * h) for w, h in sizes]
        s["batch"] = V.Batch(len(sizes))
        move = np.random.default_rng([seed, 2]).uniform(-0.02, 0.02, (len(sizes), 2))
        s["views"] = [V.view(V.VAFR_VIEW_VAFR, s["scene"], cam, V.gaze(g[0] + m[0] * w, g[1] + m[1] * h), V.shading(),
                             layout=L, lp_rgba=lp, img_rgba=img)
                      for (w, h), g, m, L, lp, img in zip(sizes, gazes, move, s["layouts"], s["lp"], s["img"])]
        return s
    w, h = case["w"], case["h"]
    s["gaze"] = V.gaze(*_gaze(w, h, seed))
    s["img"] = _rgba(w * h)
    if kind != "full":
        s["layout"] = L = _layout(case, w, h)
    if kind in ("map", "densemap"):
        s["lp"] = _random_lp(L.n_texels, seed)
        return s
    s["scene"], _, _ = _scene(case, seed)
    left, right = _cameras(case, seed)
    s["cam"], s["cam2"] = V.camera(left), V.camera(right)
    s["shading"] = V.shading()
    if kind == "full":
        s["disp"], s["id"] = V.display(w, h, I.FOV), _ids(w * h)
        return s
    s["lp"] = _rgba(L.n_texels)
    if kind in ("eye", "dense", "rep"):
        s["id"] = _ids(L.n_texels)
    if kind == "fxaa":
        V.vafr_shade_lp(s["scene"], s["cam"], s["gaze"], s["shading"], L, s["lp"])
        s["aa"] = _rgba(L.n_texels)
        del s["img"]
    if kind in ("frame", "rep"):
        s["lp2"], s["img2"] = _rgba(L.n_texels), _rgba(w * h)
    if kind == "rep":
        s["id2"] = _ids(L.n_texels)
        s["work"] = torch.empty(V.rep_workspace_bytes(L), device="cuda", dtype=torch.uint8)
    if kind == "frame":
        sh = s["shading"] if case["bounces"] < 0 else V.shading(mode=V.VAFR_SHADE_PATH, bounces=case["bounces"],
                                                                seed=seed, frame=seed & 0xffff)
        s["batch"] = V.Batch(2)
        s["views"] = [V.view(V.VAFR_VIEW_VAFR, s["scene"], c, s["gaze"], sh, layout=L, lp_rgba=lp, img_rgba=img)
                      for c, lp, img in ((s["cam"], s["lp"], s["img"]), (s["cam2"], s["lp2"], s["img2"]))]
    return s


# --------------------------------------------------------------------- run

def run(s):
    kind = s["kind"]
    if kind == "map":
        V.vafr_reconstruct(s["layout"], s["gaze"], s["lp"], s["img"])
        return s["img"]
    if kind == "densemap":
        (V.lmfr_reconstruct if s["method"] == "lmfr" else V.lafr_reconstruct)(s["layout"], s["gaze"], s["lp"],
                                                                              s["img"])
        return s["img"]
    if kind == "eye":
        V.vafr_shade_lp(s["scene"], s["cam"], s["gaze"], s["shading"], s["layout"], s["lp"], s["id"])
        V.vafr_reconstruct(s["layout"], s["gaze"], s["lp"], s["img"])
        return s["lp"], s["img"], s["id"]
    if kind == "dense":
        lmfr = s["method"] == "lmfr"
        (V.lmfr_shade_lp if lmfr else V.lafr_shade_lp)(s["scene"], s["cam"], s["gaze"], s["shading"], s["layout"],
                                                       s["lp"], s["id"])
        (V.lmfr_reconstruct if lmfr else V.lafr_reconstruct)(s["layout"], s["gaze"], s["lp"], s["img"])
        return s["lp"], s["img"], s["id"]
    if kind == "full":
        V.full_shade(s["scene"], s["cam"], s["disp"], s["shading"], s["img"], s["id"])
        return s["img"], s["id"]
    if kind == "frame":
        s["batch"].run(s["views"])
        return s["lp"], s["img"], s["lp2"], s["img2"]
    if kind == "mix":
        s["batch"].run(s["views"])
        return s["lp"], s["img"]
    if kind == "fxaa":
        V.vafr_fxaa_lp(s["layout"], s["lp"], s["aa"])
        return s["aa"]
    if kind == "rep":
        V.vafr_shade_lp_rep(s["scene"], s["cam"], s["cam2"], s["gaze"], s["shading"], s["layout"], s["lp"], s["lp2"],
                            s["work"], s["id"], s["id2"])
        V.vafr_reconstruct(s["layout"], s["gaze"], s["lp"], s["img"])
        V.vafr_reconstruct(s["layout"], s["gaze"], s["lp2"], s["img2"])
        return s["lp"], s["img"], s["lp2"], s["img2"], s["id"], s["id2"]
    raise ValueError(kind)


# -------------------------------------------------------------------- work

# Arithmetic a ray cannot do without: descending a tree over n triangles four
# ways at a time is log4(n) nodes, a node is four boxes of 6 multiply-adds and
# 5 comparisons, and one triangle test is 39 operations; shading is 40 more.
def _ray_flops(n_tris):
    return 4.0 * 17.0 * max(1.0, math.log(max(2, n_tris), 4.0)) + 39.0 + 40.0


def _tris(case):
    if case["scene"] == "soup":
        return case["size"]
    return case["size"] * case["size"] + 320 * (case["size"] * case["size"] // 4096)


def _texels(case, w, h):
    if "method" in case:
        d = DELTA[case["method"]]
        return round(w / d) * round(h / d)
    return {"standard": 1063314, "cap9": 876823, "cap18": 1018942, "aniso": 714874}[case.get("acuity", "standard")]


def work(case):
    kind = case["kind"]
    if kind == "mix":
        sizes, _ = I.batch_views(case["views"], seed=case["mixseed"])
        texels, pixels, rays = 1063314 * len(sizes), sum(w * h for w, h in sizes), 2.0 * 1063314 * len(sizes)
        return {"bytes": 16.0 * pixels + 32.0 * texels, "flops": rays * _ray_flops(_tris(case)) + 60.0 * pixels}
    w, h = case["w"], case["h"]
    pixels = w * h
    if kind == "full":
        return {"bytes": 20.0 * pixels, "flops": 2.0 * pixels * _ray_flops(_tris(case))}
    texels = _texels(case, w, h)
    if kind in ("map", "densemap"):
        # four taps a pixel: a small display does not touch every texel
        return {"bytes": 16.0 * (pixels + min(texels, 4 * pixels)), "flops": 60.0 * pixels}
    if kind == "fxaa":
        return {"bytes": 32.0 * texels, "flops": 60.0 * texels}
    if kind in ("eye", "dense"):
        # the LP buffer is written and read back, the ids written
        return {"bytes": 16.0 * pixels + 36.0 * texels,
                "flops": 2.0 * texels * _ray_flops(_tris(case)) + 60.0 * pixels}
    if kind == "rep":
        return {"bytes": 32.0 * pixels + 72.0 * texels,
                "flops": 2.0 * texels * _ray_flops(_tris(case)) + 120.0 * pixels}
    rays = 2.0 * (1 + max(0, case["bounces"]))
    return {"bytes": 32.0 * pixels + 64.0 * texels,
            "flops": 2.0 * texels * rays * _ray_flops(_tris(case)) + 120.0 * pixels}


# ------------------------------------------------- the same in 64 bits

def _columns():
    """The standard curve's columns: eccentricity (degrees) and rows of each,
    and u(e) as a function on the GPU."""
    m, b, c, u = [], [], [], [0.0]
    for k in range(len(ECC) - 1):
        m0, m1 = 1.0 / CPD[k], 1.0 / CPD[k + 1]
        m.append((m1 - m0) / (ECC[k + 1] - ECC[k]))
        b.append(m0 - m[k] * ECC[k])
        c.append(u[k] - 2.0 * math.log(m0) / m[k])
        u.append(2.0 * math.log(m1) / m[k] + c[k])
    n_cols = math.ceil(u[-1])
    e, rows = [], []
    for i in range(n_cols):
        k = max(q for q in range(len(m)) if i + 0.5 >= u[q])
        e.append((math.exp((i + 0.5 - c[k]) * m[k] * 0.5) - b[k]) / m[k])
        rows.append(max(1, math.ceil(360.0 * math.sin(math.radians(2.0 * e[i])) / (m[k] * e[i] + b[k]))))
    mt, bt, ct = (torch.tensor(x, dtype=torch.float64, device="cuda") for x in (m, b, c))
    edges = torch.tensor(ECC[1:-1], dtype=torch.float64, device="cuda")

    def u_of(ecc):
        k = torch.bucketize(ecc, edges, right=True)
        return 2.0 * torch.log(mt[k] * ecc + bt[k]) / mt[k] + ct[k]

    return e, rows, u_of


def _pitch(w, h):
    return 2.0 * math.tan(math.radians(I.FOV[0] / 2)) / w, 2.0 * math.tan(math.radians(I.FOV[1] / 2)) / h


def _blend(lp, off, rows, i0, i1, wt, turns):
    out = 0.0
    for i, wi in ((i0, 1.0 - wt), (i1, wt)):
        n = rows[i].double()
        sp = turns * n - 0.5
        j = torch.floor(sp)
        t = (sp - j)[:, None]
        j0, j1 = torch.remainder(j, n).long(), torch.remainder(j + 1.0, n).long()
        out = out + wi[:, None] * ((1.0 - t) * lp[off[i] + j0] + t * lp[off[i] + j1])
    return out


def _map64(case, seed, lp):
    """The display image of LP buffer lp (FP64)."""
    w, h = case["w"], case["h"]
    gx, gy = _gaze(w, h, seed)
    img = torch.empty((w * h, 4), dtype=torch.float64, device="cuda")
    method = case.get("method")
    if method is None:
        px, py = _pitch(w, h)
        _, rows, u_of = _columns()
        rows = torch.tensor(rows, device="cuda")
        n_cols = len(rows)
    else:
        px = py = 1.0
        n_cols, n_rows = round(w / DELTA[method]), round(h / DELTA[method])
        rows = torch.full((n_cols,), n_rows, device="cuda")
        big_l = math.log(max(math.hypot(cx - gx, cy - gy) for cx in (0, w) for cy in (0, h)))
    off = torch.cumsum(rows, 0) - rows
    for p in range(0, w * h, 1 << 21):
        k = torch.arange(p, min(w * h, p + (1 << 21)), device="cuda")
        dx = ((k % w).double() + 0.5 - gx) * px
        dy = (torch.div(k, w, rounding_mode="floor").double() + 0.5 - gy) * py
        r = torch.hypot(dx, dy)
        if method is None:
            u = u_of(torch.rad2deg(torch.atan(r)))
        else:
            z = torch.log(r.clamp(min=1.0)) / big_l
            if method == "lmfr":
                u = z ** 4 * n_cols
            else:   # both pieces of the two-piece kernel
                zef = math.log(math.tan(math.radians(4.89)) / _pitch(w, h)[1]) / big_l
                fa = 1.0 - math.log((V.LAFR_ALPHA * zef) ** (1 - V.LAFR_A) / (1 - V.LAFR_A)) / math.log(zef)
                uef = (zef * (1.0 - fa)) ** (1.0 / fa)
                za = (1.0 / z.clamp(min=zef) - 1.0 / zef) / (1.0 / zef - 1.0)
                outer = ((2.0 * torch.acos(za.clamp(-1.0, 1.0)) - math.pi) / math.pi).clamp(min=0.0)
                outer = outer ** (V.LAFR_BETA / 0.7) * (1.0 - uef) + uef
                u = torch.where(z <= zef, (z * (1.0 - fa)) ** (1.0 / fa), outer) * n_cols
        a = u.clamp(0.5, n_cols - 0.5) - 0.5
        i0 = a.long().clamp(max=n_cols - 1)
        turns = torch.remainder(torch.atan2(dy, dx) / (2.0 * math.pi), 1.0)
        img[k] = _blend(lp, off, rows, i0, (i0 + 1).clamp(max=n_cols - 1), a - i0.double(), turns)
    return img


def _hit64(tri, org, d, nearest):
    """Nearest hit (t, triangle) of rays org + t d with t > 0, or whether any
    triangle is hit, by testing every triangle."""
    v0, e1, e2 = tri
    t_best = torch.full((d.shape[0],), math.inf, dtype=torch.float64, device="cuda")
    k_best = torch.zeros(d.shape[0], dtype=torch.int64, device="cuda")
    step = max(1, (1 << 25) // v0.shape[0])
    for p in range(0, d.shape[0], step):
        o, q = org[p:p + step, None, :], d[p:p + step, None, :]
        pv = torch.linalg.cross(q.expand(-1, v0.shape[0], -1), e2[None].expand(q.shape[0], -1, -1))
        det = (pv * e1).sum(-1)
        s = o - v0[None]
        u = (s * pv).sum(-1) / det
        del pv
        qv = torch.linalg.cross(s, e1[None].expand(s.shape[0], -1, -1))
        del s
        v = (qv * q).sum(-1) / det
        t = (qv * e2).sum(-1) / det
        t = torch.where((u >= 0) & (v >= 0) & (u + v <= 1) & (t > 0), t, math.inf)
        t_best[p:p + step], k_best[p:p + step] = t.min(1)
    return (t_best, k_best) if nearest else t_best < math.inf


def _albedo64(ids):
    m = 0xffffffff
    x = (ids * 747796405 + 2891336453) & m
    x = (((x >> ((x >> 28) + 4)) ^ x) * 277803737) & m
    x = (x >> 22) ^ x
    return torch.stack([0.2 + 0.7 * ((x >> s) & 255).double() / 255.0 for s in (0, 8, 16)], 1)


def _shade64(case, seed):
    """The LP buffer of a soup's left eye."""
    _, verts, tris = _scene(case, seed)
    e, rows, _ = _columns()
    dev = {"dtype": torch.float64, "device": "cuda"}
    p = torch.tensor(verts[tris], **dev)
    tri = (p[:, 0], p[:, 1] - p[:, 0], p[:, 2] - p[:, 0])
    n = torch.tensor(rows, device="cuda")
    col = torch.repeat_interleave(torch.arange(len(rows), device="cuda"), n)
    j = torch.arange(int(n.sum()), device="cuda") - (torch.cumsum(n, 0) - n)[col]
    th = 2.0 * math.pi * (j.double() + 0.5) / n[col].double()
    rho = torch.tan(torch.deg2rad(torch.tensor(e, **dev)))[col]
    w, h = case["w"], case["h"]
    (px, py), (gx, gy) = _pitch(w, h), _gaze(w, h, seed)
    fx, fy = (gx - 0.5 * w) * px + rho * torch.cos(th), (gy - 0.5 * h) * py + rho * torch.sin(th)
    eye, right, up, fwd = torch.tensor(_cameras(case, seed)[0].reshape(4, 3), **dev)
    d = fx[:, None] * right - fy[:, None] * up + fwd
    t, k = _hit64(tri, eye.expand(d.shape[0], 3), d, True)
    hit = torch.nonzero(t < math.inf)[:, 0]
    out = torch.tensor([0.05, 0.05, 0.08, 1.0], **dev).repeat(d.shape[0], 1)
    pos = eye + t[hit, None] * d[hit]
    nrm = torch.linalg.cross(tri[1][k[hit]], tri[2][k[hit]])
    nrm = nrm / torch.linalg.norm(nrm, dim=1, keepdim=True)
    nrm = torch.where(((nrm * d[hit]).sum(1) > 0)[:, None], -nrm, nrm)
    light = torch.tensor([0.3, 1.0, -0.5], **dev)
    light = light / torch.linalg.norm(light)
    ndl = (nrm * light).sum(1).clamp(min=0.0)
    org = pos + nrm * 1e-4 * (1.0 + pos.abs().max(1, keepdim=True).values)
    lit = torch.nonzero(ndl > 0)[:, 0]
    dark = _hit64(tri, org[lit], light.expand(len(lit), 3), False)
    ndl[lit[dark]] = 0.0
    out[hit, :3] = _albedo64(k[hit]) * (0.1 + ndl[:, None])
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("map", "densemap"):
        return _map64(case, seed, _random_lp(_texels(case, case["w"], case["h"]), seed).double())
    if kind == "eye" and case["scene"] == "soup" and case["acuity"] == "standard" and case["size"] <= 4096:
        lp = _shade64(case, seed)
        return lp, _map64(case, seed, lp), None
    # the larger scenes take too long to ray-cast against every triangle
    return None
