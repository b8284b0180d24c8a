"""The work a user of the depth-of-field library has it do, as cases to time.

A case names one call of a public entry point with its sizes and options:

  frame      one hybrid depth-of-field frame on the previous frame's history
  batch      one step of several sessions, one frame each, as one batch
  build      the acceleration structure of a scene (every frame of a scene that moves)
  gbuffer    the pinhole G-buffer of a view
  rays       closest hits of the caller's own rays (picking, focus queries, probes)
  reference  the fully ray-traced ground truth of a view

Scenes are the repository's synthetic families ("small": boxes and bars, 866
triangles; "grass": spheres behind a grass band; "fence": a box city behind a
chain-link fence) at any triangle count.  `prepare` makes what a program holds
before the call -- the scene on the device with its tree, the G-buffer, the
previous frame's history, the frame's buffers -- and `run` is one pass.

The traversal's own counters (node visits, triangle tests) describe how the
library worked and not what it computed, so they are not among the outputs;
the numbers of masked pixels and rays are those of the returned mask.
"""

import dataclasses
import math

import numpy as np
import torch

from paper_2210_06158_amd import dof, synth

MODES = {"adaptive": synth.MASK_ADAPTIVE, "fixed": synth.MASK_FIXED, "dilate": synth.MASK_DILATE}
GRASS_TRIS, FENCE_TRIS = 1183042, 1960002


def listed():
    return [
        # the smallest interactive view (a preview or thumbnail): launches and latency count
        dict(name="frame 256x256", kind="frame", scene="small", tris=866, split=2, width=256, height=256, m=4,
             mask="adaptive", blades=0, polygon=False, taa=0, fp16=False, frame=1),
        # an odd window size with every option on: hexagonal bokeh, dilated mask, all TAA stages, jitter, FP32 images
        dict(name="frame 1366x766 options", kind="frame", scene="grass", tris=300000, split=2, width=1366, height=766,
             m=30, mask="dilate", blades=6, polygon=True, taa=7, fp16=False, frame=20),
        # the ordinary frame: 1080p, 1.18 M triangles, 8 rays per masked pixel
        dict(name="frame 1920x1080", kind="frame", scene="grass", tris=GRASS_TRIS, split=3, width=1920, height=1080,
             m=8, mask="adaptive", blades=0, polygon=False, taa=0, fp16=True, frame=20),
        # the largest frame: 4K through a thin out-of-focus fence, 16 rays per masked pixel
        dict(name="frame 3840x2160", kind="frame", scene="fence", tris=FENCE_TRIS, split=0, width=3840, height=2160,
             m=16, mask="adaptive", blades=6, polygon=False, taa=0, fp16=True, frame=30),
        # a server's step: eight viewers, each with a scene of its own, 720p to 1440p
        dict(name="batch of 8", kind="batch", sessions=8, tris=400000, split=3, width=0, height=0, m=8),
        # the tree of a tiny scene, as a moving scene needs it every frame
        dict(name="build 866", kind="build", scene="small", tris=866, split=2),
        # the tree of the ordinary scene
        dict(name="build 1183042", kind="build", scene="grass", tris=GRASS_TRIS, split=3),
        # the G-buffer of the smallest and of the ordinary view
        dict(name="gbuffer 256x256", kind="gbuffer", scene="small", tris=866, split=2, width=256, height=256,
             fp16=False, frame=0),
        dict(name="gbuffer 1920x1080", kind="gbuffer", scene="grass", tris=GRASS_TRIS, split=3, width=1920,
             height=1080, fp16=True, frame=20),
        # a handful of queries (what is under the cursor, the distance to focus on)
        dict(name="rays 1000", kind="rays", scene="small", tris=866, split=2, rays=1000, spread="view"),
        # a million incoherent rays in every direction (probes, occlusion baking)
        dict(name="rays 1000000", kind="rays", scene="grass", tris=GRASS_TRIS, split=2, rays=1000000,
             spread="sphere"),
        # the ground truth an image-quality check renders
        dict(name="reference 1280x720", kind="reference", scene="grass", tris=300000, split=2, width=1280, height=720,
             spp=16, blades=0, frame=20),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """An even width between lo and hi and an even height between half and all of it."""
    w = _log(rng, lo, hi)
    h = max(2, int(w * rng.uniform(0.5, 1.0)))
    return w - w % 2, h - h % 2


def _scene(rng):
    name = rng.choice(["small", "grass", "grass", "fence"])
    most = {"small": 866, "grass": GRASS_TRIS, "fence": FENCE_TRIS}[name]
    return dict(scene=name, tris=866 if name == "small" else _log(rng, 20000, most), split=rng.choice([0, 1, 2, 3]))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "batch", "build", "build", "gbuffer", "rays", "rays", "reference"])
    if kind == "batch":
        w, h = _size(rng, 320, 1920)
        return dict(kind=kind, sessions=rng.randint(2, 8), tris=_log(rng, 20000, 400000), split=rng.choice([0, 2, 3]),
                    width=w, height=h, m=_log(rng, 1, 8))
    case = dict(kind=kind, **_scene(rng))
    if kind == "frame":
        w, h = _size(rng, 128, 3840)
        h = min(h, 2160)
        m = _log(rng, 1, 30)
        m = max(1, min(m, 3840 * 2160 * 12 // (w * h)))
        blades = rng.choice([0, 0, 5, 6, 9])
        case.update(width=w, height=h, m=m, mask=rng.choice(["adaptive", "adaptive", "adaptive", "fixed", "dilate"]),
                    blades=blades, polygon=blades > 0 and rng.random() < 0.5, taa=rng.choice([0, 0, 1, 7]),
                    fp16=rng.random() < 0.7, frame=rng.randint(1, 59))
    elif kind == "gbuffer":
        w, h = _size(rng, 128, 2560)
        case.update(width=w, height=h, fp16=rng.random() < 0.7, frame=rng.randint(0, 59))
    elif kind == "rays":
        case.update(rays=_log(rng, 100, 2000000), spread=rng.choice(["view", "sphere"]))
    elif kind == "reference":
        w, h = _size(rng, 128, 1280)
        spp = _log(rng, 1, 64)
        case.update(width=w, height=h, spp=max(1, min(spp, 1280 * 720 * 16 // (w * h))), blades=rng.choice([0, 6]),
                    frame=rng.randint(0, 59))
    return case


# ---------------------------------------------------------------- inputs

def _inputs(case, seed):
    """The scene, the camera of the case's frame and of the one before, their
    lenses and the pass's parameters: made from the seed alone, on the host."""
    w, h, f = case.get("width", 256), case.get("height", 256), case.get("frame", 0)
    sd = synth.BASE_SEED + 7919 * (seed + 1)
    if case["scene"] == "small":
        scene, cam, lens, _ = synth.scene_small(seed=sd)
        cam = dataclasses.replace(cam, width=w, height=h)
        cams = [dataclasses.replace(synth.pan_camera(cam, 0.02 * k), frame=k) for k in range(60)]
        lenses = [lens] * 60
    elif case["scene"] == "grass":
        part = case["tris"] / GRASS_TRIS
        scene, cams, lens, _ = synth.scene_1080p(seed=sd, n_spheres=max(1, round(4096 * part)),
                                                 n_blades=max(1, round(50000 * part)), width=w, height=h)
        lenses = [lens] * 60
    else:
        part = case["tris"] / FENCE_TRIS
        scene, cams, lenses, _ = synth.scene_4k(seed=sd, n_boxes=max(1, round(130000 * part)),
                                                n_links=max(1, round(200000 * part)))
        cams = [dataclasses.replace(c, width=w, height=h) for c in cams]
        lenses = [dataclasses.replace(l, blades=0) for l in lenses]
    scene = dataclasses.replace(scene, leaf_split=case["split"])
    lenses = [dataclasses.replace(l, blades=case.get("blades", 0)) for l in lenses]
    if case.get("taa"):
        cams = synth.jittered(cams, seed=sd)
    p = synth.Params(m=case.get("m", 8), mask_mode=MODES[case.get("mask", "adaptive")], taa=case.get("taa", 0),
                     pp_polygon=int(case.get("polygon", False)))
    return scene, cams[f], lenses[f], cams[max(f - 1, 0)], lenses[max(f - 1, 0)], p


def _turned(scene, seed):
    """The scene with its axes permuted and mirrored, scaled by a power of two,
    its triangles listed from another one on and with albedos of its own: other
    triangles and another tree, of as many leaves (which a random scene's long
    thin triangles would change a little from seed to seed)."""
    rng = np.random.default_rng(seed)
    sign = rng.choice([-1.0, 1.0], 3) * 2.0 ** rng.integers(-2, 3)
    v = scene.verts.reshape(-1, 3, 3)[..., rng.permutation(3)] * sign.astype(np.float32)
    v = np.roll(v.reshape(-1, 9), int(rng.integers(scene.ntri)), 0)
    return dataclasses.replace(scene, verts=v, albedo=rng.random(scene.albedo.shape, np.float32))


def _rays(case, seed, cam, lens):
    """Host arrays of the caller's rays: through random points of the view, or
    from random points near the camera in every direction."""
    rng = np.random.default_rng(seed)
    n = case["rays"]
    if case["spread"] == "view":
        t = synth.half_fov_tan(lens)
        u, v = rng.uniform(-t, t, (2, n))
        d = np.asarray(cam.fwd) + u[:, None] * np.asarray(cam.right) + v[:, None] * np.asarray(cam.up)
        o = np.broadcast_to(np.asarray(cam.pos), (n, 3))
    else:
        d = rng.normal(size=(n, 3))
        o = np.asarray(cam.pos) + rng.uniform((-2.0, -0.7, 0.0), (2.0, 0.7, 4.0), (n, 3))
    return np.ascontiguousarray(o, np.float32), np.ascontiguousarray(d, np.float32)


def _built(scene):
    gs = dof.Scene(scene)
    gs.build_bvh()
    return gs


def _frame_state(gs, cam, lens, pcam, plens, p, fp16):
    """A frame's buffers with the previous frame rendered into its history."""
    fmt = dof.RGBA16F if fp16 else dof.RGBA32F
    w, h = cam.width, cam.height
    fr = dof.Frame(w, h, p, out_format=fmt)
    hist = [dof.history_alloc(w, h), dof.history_alloc(w, h)]
    fr.render(gs, pcam, plens, gs.render_gbuffer(pcam, plens, fmt=fmt), None, hist[0])
    return dict(gs=gs, frame=fr, cam=cam, lens=lens, pcam=pcam, plens=plens, hist=hist,
                gb=gs.render_gbuffer(cam, lens, fmt=fmt))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        sizes = [(case["width"], case["height"])] if case["width"] else synth.SESSION_SIZES
        part = case["tris"] / GRASS_TRIS
        items, p = [], synth.Params(m=case["m"])
        for i in range(case["sessions"]):
            w, h = sizes[i % len(sizes)]
            scene, cams, lens, _ = synth.scene_1080p(
                seed=synth.BASE_SEED + 7919 * (seed + 1) + 104729 * i, n_spheres=max(1, round(4096 * part)),
                n_blades=max(1, round(50000 * part)), width=w, height=h)
            gs = _built(dataclasses.replace(scene, leaf_split=case["split"]))
            items.append(_frame_state(gs, cams[20], lens, cams[19], lens, p, True))
        return dict(kind=kind, items=items, batch=dof.Batch(case["sessions"], p))
    if kind == "build":
        return dict(kind=kind, gs=dof.Scene(_turned(_inputs(case, 0)[0], seed)))
    scene, cam, lens, pcam, plens, p = _inputs(case, seed)
    gs = _built(scene)
    if kind == "rays":
        o, d = (torch.from_numpy(a).cuda() for a in _rays(case, seed, cam, lens))
        return dict(kind=kind, gs=gs, org=o, dir=d)
    if kind == "frame":
        return dict(kind=kind, **_frame_state(gs, cam, lens, pcam, plens, p, case["fp16"]))
    st = dict(kind=kind, gs=gs, cam=cam, lens=lens)
    if kind == "gbuffer":
        dt = torch.float16 if case["fp16"] else torch.float32
        st["images"] = (torch.empty((cam.height, cam.width, 4), dtype=dt, device="cuda"),
                        torch.empty((cam.height, cam.width), device="cuda"),
                        torch.empty((cam.height, cam.width, 4), dtype=dt, device="cuda"))
    else:
        st["spp"] = case["spp"]
    return st


def _frame_out(s):
    return dict(colour=s["frame"].colour, mask=s["frame"].mask, history=s["hist"][1])


def run(state):
    kind = state["kind"]
    if kind == "frame":
        s = state
        s["frame"].render(s["gs"], s["cam"], s["lens"], s["gb"], s["hist"][0], s["hist"][1], prev_cam=s["pcam"],
                          prev_lens=s["plens"])
        return _frame_out(s)
    if kind == "batch":
        state["batch"].set([s["frame"].item(s["gs"], s["cam"], s["lens"], s["gb"], s["hist"][0], s["hist"][1],
                                            prev_cam=s["pcam"], prev_lens=s["plens"]) for s in state["items"]])
        state["batch"].run()
        return [_frame_out(s) for s in state["items"]]
    if kind == "build":
        state["gs"].build_bvh()
        v = state["gs"].bvh_view()
        # node and triangle records hold indices beside their planes: as bits
        return dict(v, nodes=v["nodes"].view(torch.int32), tris=v["tris"].view(torch.int32))
    if kind == "gbuffer":
        return state["gs"].render_gbuffer_into(state["cam"], state["lens"], *state["images"])
    if kind == "rays":
        return state["gs"].trace_rays(state["org"], state["dir"])
    return state["gs"].render_reference(state["cam"], state["lens"], state["spp"])


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    """Bytes of the inputs read once and the outputs written once; operations
    of a closest hit as one descent of the tree (24 per pair of boxes) and one
    triangle test (40), and of the two 81-tap filters.  A frame's mask decides
    how many rays it traces: 45 % of the budget is taken, what the scenes'
    frames trace on average."""
    kind = case["kind"]
    if kind == "batch":
        sizes = [(case["width"], case["height"])] if case["width"] else synth.SESSION_SIZES
        one = [work(dict(kind="frame", scene="grass", tris=case["tris"], width=w, height=h, m=case["m"], taa=0,
                         fp16=True)) for w, h in (sizes[i % len(sizes)] for i in range(case["sessions"]))]
        return {k: sum(x[k] for x in one) for k in ("bytes", "flops")}
    per_ray = 24 * math.log2(max(case["tris"], 2)) + 40
    if kind == "build":
        # vertices, albedos and offsets in; per leaf its triangle, albedo, key, id, two nodes and two links out
        return dict(bytes=case["tris"] * (36 + 12 + 4 + 48 + 16 + 8 + 4 + 64 + 32 + 8), flops=case["tris"] * 60)
    if kind == "rays":
        return dict(bytes=case["rays"] * 32, flops=case["rays"] * per_ray)
    px = case["width"] * case["height"]
    if kind == "reference":
        return dict(bytes=px * 16, flops=px * case["spp"] * per_ray)
    image = 8 if case["fp16"] else 16
    if kind == "gbuffer":
        return dict(bytes=px * (2 * image + 4), flops=px * per_ray)
    half = px // 4
    planes = (16 if case["taa"] & 1 else 0) + (16 if case["taa"] & 2 else 0) + (4 if case["taa"] & 4 else 0)
    return dict(bytes=px * (image + 4 + image / 4 + image + 2 * planes) + half * (2 * 52 + 1),
                flops=0.45 * half * case["m"] * per_ray + half * 81 * (14 + 50))


# ---------------------------------------------------------------- the same in 64 bits

MOST_PAIRS = 2e10   # ray-triangle pairs that brute force gets through in a few seconds
SQRT2 = 1.41421356237


def _t(v):
    return torch.as_tensor(np.asarray(v, np.float32), device="cuda").double()


class _World:
    """A scene in 64 bits: closest hits by testing every triangle."""

    def __init__(self, scene):
        self.v = _t(scene.verts).reshape(-1, 3, 3)
        self.albedo = _t(scene.albedo)
        self.light, self.rad, self.amb, self.sky = (_t(getattr(scene, k)) for k in
                                                    ("light_dir", "light_rad", "ambient", "sky"))

    def hits(self, o, d):
        """(triangle or -1, distance or inf) of each ray (Moeller and Trumbore 1997)."""
        v0, e1, e2 = self.v[:, 0], self.v[:, 1] - self.v[:, 0], self.v[:, 2] - self.v[:, 0]
        n, ids, ts = torch.linalg.cross(e1, e2), [], []
        step = max(1, 8_000_000 // len(v0))
        for k in range(0, len(o), step):
            oo, dd = o[k:k + step], d[k:k + step]
            det = dd @ n.T
            # (o - v0) . n and the two edge coordinates, from per-triangle and per-ray parts
            m = torch.linalg.cross(oo, dd)
            t = ((v0 * n).sum(1) - oo @ n.T) / det
            u = -(m @ e2.T - dd @ torch.linalg.cross(e2, v0).T) / det
            w = (m @ e1.T - dd @ torch.linalg.cross(e1, v0).T) / det
            t = torch.where((u >= 0) & (w >= 0) & (u + w <= 1) & (t > 0) & (det != 0), t, math.inf)
            best, at = t.min(1)
            ids.append(torch.where(best < math.inf, at, -1))
            ts.append(best)
        return torch.cat(ids), torch.cat(ts)

    def shade(self, ids, d):
        """Lambert colour and normal facing the ray; the sky's colour on a miss."""
        v = self.v[ids.clamp(min=0)]
        n = torch.linalg.cross(v[:, 1] - v[:, 0], v[:, 2] - v[:, 0])
        n = n / n.norm(dim=1, keepdim=True)
        n = torch.where((n * d).sum(1, keepdim=True) > 0, -n, n)
        ndl = (-(n * self.light).sum(1, keepdim=True)).clamp(min=0)
        c = self.albedo[ids.clamp(min=0)] * (self.rad * ndl + self.amb)
        hit = (ids >= 0)[:, None]
        return torch.where(hit, c, self.sky), torch.where(hit, n, 0.0)


class _View:
    """A camera and lens: the thin lens' constants and the pixels' directions."""

    def __init__(self, cam, lens, jitter=True):
        f, n, d, ws = (float(np.float32(x)) for x in (lens.focal, lens.fnum, lens.focus, lens.sensor))
        self.w, self.h, self.cam, self.lens, self.d = cam.width, cam.height, cam, lens, d
        self.pos, self.right, self.up, self.fwd = (_t(getattr(cam, k)) for k in ("pos", "right", "up", "fwd"))
        self.tx = ws * (d - f) / (2 * f * d)
        self.ty = self.tx * self.h / self.w
        self.a = f / n
        self.cock = self.a * f / (d - f) * self.w / ws
        g = SQRT2 * (d - f) * ws / self.w
        self.znb = self.a * f * d / (self.a * f + g)
        self.ramp = 2 * (d - self.znb)
        jx, jy = (float(np.float32(x)) for x in (cam.jitter if jitter else (0.0, 0.0)))
        self.ju, self.jv = jx * 2 / self.w, jy * 2 / self.h

    def dirs(self, w, h):
        x = torch.arange(w, device="cuda", dtype=torch.float64)[None, :]
        y = torch.arange(h, device="cuda", dtype=torch.float64)[:, None]
        u = ((x + 0.5) * 2 / w - 1 + self.ju) * self.tx
        v = ((1 - (y + 0.5) * 2 / h) - self.jv) * self.ty
        return (self.fwd + u[..., None] * self.right + v[..., None] * self.up).reshape(-1, 3)

    def coc(self, z):
        return self.cock * (1 - self.d / z).abs()

    def lens_rays(self, q, k, w, h):
        """Ray k of pixel q of a w x h grid (counter-hashed lens point)."""
        seed = _pcg(_pcg(_pcg(torch.tensor(self.cam.seed & 0xffffffff, device="cuda")) ^ self.cam.frame) ^ q)
        lx, ly = torch.zeros(len(q), device="cuda", dtype=torch.float64), torch.zeros(len(q), device="cuda", dtype=torch.float64)
        todo = torch.ones(len(q), device="cuda", dtype=torch.bool)
        nb = self.lens.blades
        for att in range(32):
            a = _pcg(seed ^ ((k << 8) | att))
            x, y = ((b >> 8).double() / 8388608 - 1 for b in (a, _pcg(a)))
            if nb < 3:
                ok = x * x + y * y < 1
            else:
                ok = torch.ones_like(todo)
                for i in range(nb):
                    th = self.lens.blade_rot + math.pi / nb + 2 * math.pi * i / nb
                    ok &= x * math.cos(th) + y * math.sin(th) <= math.cos(math.pi / nb)
            lx, ly = torch.where(todo & ok, x, lx), torch.where(todo & ok, y, ly)
            todo &= ~ok
        pf = self.pos + self.dirs(w, h)[q] * self.d
        o = self.pos + self.a / 2 * (lx[:, None] * self.right + ly[:, None] * self.up)
        d = pf - o
        return o, d / d.norm(dim=1, keepdim=True)


def _pcg(v):
    """The PCG hash of 32-bit values held in 64 bits."""
    s = (v * 747796405 + 2891336453) & 0xffffffff
    w = (((s >> ((s >> 28) + 4)) ^ s) * 277803737) & 0xffffffff
    return ((w >> 22) ^ w) & 0xffffffff


def _gbuffer64(world, view):
    d = view.dirs(view.w, view.h)
    d = d / d.norm(dim=1, keepdim=True)
    o = view.pos.expand_as(d)
    ids, t = world.hits(o, d)
    c, n = world.shade(ids, d)
    z = torch.where(ids >= 0, t * (d @ view.fwd), math.inf)
    hw = (view.h, view.w)
    one = torch.ones_like(c[:, :1])
    return (torch.cat([c, one], 1).reshape(*hw, 4), z.reshape(hw), torch.cat([n, 0 * one], 1).reshape(*hw, 4))


def _at(img, y, x):
    """img at integer positions clamped to its edges."""
    return img[y.clamp(0, img.shape[0] - 1), x.clamp(0, img.shape[1] - 1)]


def _bilinear(img, x, y):
    x0, y0 = x.floor(), y.floor()
    fx, fy = (x - x0)[..., None], (y - y0)[..., None]
    x0, y0 = x0.long(), y0.long()
    top = torch.lerp(_at(img, y0, x0), _at(img, y0, x0 + 1), fx)
    return torch.lerp(top, torch.lerp(_at(img, y0 + 1, x0), _at(img, y0 + 1, x0 + 1), fx), fy)


def _around(img, r=1):
    """The (2r + 1)^2 neighbours of every pixel, clamped to the edges, in row order."""
    h, w = img.shape[:2]
    y = torch.arange(h, device=img.device)[:, None]
    x = torch.arange(w, device=img.device)[None, :]
    return [_at(img, y + j, x + i) for j in range(-r, r + 1) for i in range(-r, r + 1)]


def _filter(img, ky, kx):
    """Separable 5- or 3-tap filter, clamped to the edges."""
    r = len(kx) // 2
    y = torch.arange(img.shape[0], device=img.device)[:, None]
    x = torch.arange(img.shape[1], device=img.device)[None, :]
    img = sum(k * _at(img, y, x + i - r) for i, k in enumerate(kx))
    return sum(k * _at(img, y + i - r, x) for i, k in enumerate(ky))


def _taps():
    """The centre and four rings of 8, 16, 24 and 32 taps: (x, y, radius)."""
    out = [(0.0, 0.0, 0.0)]
    for k in range(1, 5):
        out += [(float(np.float32(k / 4 * math.cos(2 * math.pi * j / (8 * k)))),
                 float(np.float32(k / 4 * math.sin(2 * math.pi * j / (8 * k)))), k / 4) for j in range(8 * k)]
    return out


def _luma(c):
    return 0.2126 * c[..., 0] + 0.7152 * c[..., 1] + 0.0722 * c[..., 2]


def _reproject(prev, p, direction, w, h):
    """Texel of the previous view's w x h grid that sees p (or a direction); -1 outside."""
    e = torch.where(direction[..., None], p, p - prev.pos)
    ex, ey, ez = e @ prev.right, e @ prev.up, e @ prev.fwd
    sx = (ex / ez / prev.tx + 1) / 2 * w
    sy = (1 - ey / ez / prev.ty) / 2 * h
    ok = (ez > 0) & (sx >= 0) & (sx < w) & (sy >= 0) & (sy < h)
    return torch.where(ok, torch.where(ok, sy, 0).long() * w + torch.where(ok, sx, 0).long(), -1)


def _frame64(world, view, prev, hist, gbuffer, p):
    """One frame of the pass without its optional stages: colour, mask and the
    history planes (near rgb + hit ratio, far rgb + age, CoCs + luma moments,
    variance).  hist: the previous frame's planes or None."""
    H, W, hh, hw = view.h, view.w, view.h // 2, view.w // 2
    colour, depth, normal = gbuffer
    sat = lambda x: torch.nan_to_num(x, nan=0.0).clamp(0, 1)  # noqa: E731
    d = view.d
    # half resolution: the quad's nearest depth, its normal, the mean colour, signed radius
    quad = lambda a: [a[j::2, i::2] for j in (0, 1) for i in (0, 1)]  # noqa: E731
    z, nrm = depth[0::2, 0::2], normal[0::2, 0::2]
    for zk, nk in zip(quad(depth)[1:], quad(normal)[1:]):
        nrm, z = torch.where((zk < z)[..., None], nk, nrm), torch.where(zk < z, zk, z)
    col = sum(quad(colour[..., :3])) / 4
    r = (view.coc(z) / 4).clamp(max=p.r_max)
    r = torch.where(z < d, -r, r)
    # largest radius of the 16 x 16 tiles and of their neighbourhood
    th, tw = -(-hh // 16), -(-hw // 16)
    pad = torch.nn.functional.pad(r.abs(), (0, tw * 16 - hw, 0, th * 16 - hh))
    tile = pad.reshape(th, 16, tw, 16).amax((1, 3))
    D = math.ceil(p.r_max / 16)
    tile = torch.nn.functional.max_pool2d(tile[None, None], 2 * D + 1, 1, D)[0, 0]
    Rn = tile.repeat_interleave(16, 0).repeat_interleave(16, 1)[:hh, :hw]
    y = torch.arange(hh, device="cuda")[:, None].expand(hh, hw)
    x = torch.arange(hw, device="cuda")[None, :].expand(hh, hw)
    xd, yd = x.double(), y.double()
    # prefilter
    sp = (Rn / 4).clamp(min=SQRT2) / 2
    cr = torch.cat([col, r[..., None]], 2)
    acc = sw = 0.0
    for dy in (-1, 0, 1):
        for dx in (-1, 0, 1):
            v = _bilinear(cr, xd + dx * sp, yd + dy * sp)
            w = 1 / (1 + (v[..., 3] - r).abs())
            acc, sw = acc + w[..., None] * v[..., :3], sw + w
    pre = acc / sw[..., None]
    # gather
    tex = torch.cat([pre, r.abs()[..., None], z[..., None], (_luma(pre) > p.l_spec).double()[..., None]], 2)
    acc, sw, ss = torch.zeros_like(pre), torch.zeros_like(z), torch.zeros_like(z)
    for ox, oy, frac in _taps():
        v = _at(tex, (yd + oy * Rn + 0.5).floor().long(), (xd + ox * Rn + 0.5).floor().long())
        dist = Rn * frac
        alpha = 1 / v[..., 3].clamp(min=0.5) ** 2
        w = torch.where(r.abs() > dist, alpha, alpha * (1 - sat((v[..., 4] - z) / p.depth_range)))
        w = torch.where(v[..., 3] > dist, w, 0.0)
        acc, sw, ss = acc + w[..., None] * v[..., :3], sw + w, ss + w * v[..., 5]
    some = sw > 0
    gat = torch.where(some[..., None], torch.cat([acc, ss[..., None]], 2) / sw.clamp(min=1e-300)[..., None],
                      torch.cat([pre, torch.zeros_like(z)[..., None]], 2))
    pp = torch.cat([torch.stack(_around(gat[..., :3])).median(0).values, gat[..., 3:]], 2)
    # mask
    g5 = (0.0625, 0.25, 0.375, 0.25, 0.0625)
    F = _filter(torch.cat([(d / z)[..., None], nrm[..., :3]], 2), g5, g5)
    sm, dv = (1, 4, 6, 4, 1), (-1, -2, 0, 2, 1)
    e = (_filter(F, sm, dv) / 128) ** 2 + (_filter(F, dv, sm) / 128) ** 2
    xx = (e[..., 0].sqrt() + e[..., 1:].sum(2).sqrt()) * p.s
    xn = sat(1 - 1 / (xx + 1))
    dirs = view.dirs(hw, hh).reshape(hh, hw, 3)
    pn = torch.full((hh, hw), -1, device="cuda")
    if hist is not None:
        sky = ~(z < math.inf)
        pn = _reproject(prev, torch.where(sky[..., None], dirs, view.pos + torch.where(sky, 0, z)[..., None] * dirs),
                        sky, hw, hh)
        pn = torch.where((pn >= 0) & (hist["B"].reshape(-1, 4)[pn.clamp(min=0), 3] > 0), pn, -1)
        var = torch.where(pn >= 0, hist["D"].reshape(-1)[pn.clamp(min=0)], 0.0)
    else:
        var = torch.zeros_like(z)
    cnt = (sat(xn + var * p.var_mask_w) * p.m + 0.5).floor().long()
    cnt = torch.maximum(cnt, ((z < d) & (view.coc(z) > SQRT2)).long()).clamp(max=p.m)
    if p.mask_mode == synth.MASK_FIXED:
        cnt = torch.where(cnt > 0, p.m, 0)
    # thin-lens rays of the masked pixels
    q = cnt.reshape(-1).nonzero()[:, 0]
    n = cnt.reshape(-1)[q]
    slot = torch.repeat_interleave(torch.arange(len(q), device="cuda"), n)
    k = torch.arange(len(slot), device="cuda") - (n.cumsum(0) - n)[slot]
    o, dr = view.lens_rays(q[slot], k, hw, hh)
    ids, t = world.hits(o, dr)
    hit = ids >= 0
    rc, _ = world.shade(ids, dr)
    P = o + torch.where(hit, t, 0.0)[:, None] * dr
    hz = torch.where(hit, (P - view.pos) @ view.fwd, math.inf)
    w = torch.where(hit, sat(0.5 + (d - hz) / view.ramp), 0.0)
    cz = view.coc(hz)

    def total(v):
        out = torch.zeros((hh * hw,) + v.shape[1:], device="cuda", dtype=torch.float64)
        return out.index_add_(0, q[slot], v).reshape((hh, hw) + v.shape[1:])

    def mean(s, c):
        c = c[..., None] if s.dim() > c.dim() else c
        return torch.where(c > 0, s / torch.where(c > 0, c, 1.0), 0.0)
    N, nf = total(w), total(1 - w)
    near, far = mean(total(w[:, None] * rc), N), mean(total((1 - w)[:, None] * rc), nf)
    cN, cF = mean(total(w * cz), N), mean(total((1 - w) * cz), nf)
    hcur = mean(N, cnt.double())
    fw = total(torch.where(hit, 1 - w, 0.0))
    fp = mean(total(torch.where(hit, 1 - w, 0.0)[:, None] * P), fw)
    # temporal accumulation; a missing far position from its valid neighbours
    on = cnt > 0
    have = on & (fw > 0)
    around = _inside_around(torch.cat([fp, torch.ones_like(z)[..., None]], 2) * have[..., None])
    fpos = torch.where(have[..., None], fp, mean(around[..., :3], around[..., 3]))
    fvalid = have | (around[..., 3] > 0)
    pf = torch.full_like(pn, -1)
    motion = False
    zero = torch.zeros((hh, hw, 4), device="cuda", dtype=torch.float64)
    hA = hB = hC = fB = fC = zero
    if hist is not None:
        pf = _reproject(prev, fpos, torch.zeros_like(on), hw, hh)
        A, B, C = (hist[i].reshape(-1, 4) for i in "ABC")
        pf = torch.where(fvalid & (pf >= 0) & (B[pf.clamp(min=0), 3] > 0), pf, -1)
        hA, hB, hC = (torch.where((pn >= 0)[..., None], v[pn.clamp(min=0)], 0.0) for v in (A, B, C))
        fB, fC = (torch.where((pf >= 0)[..., None], v[pf.clamp(min=0)], 0.0) for v in (B, C))
        motion = (view.cam.pos, view.cam.right, view.cam.up, view.cam.fwd, view.lens) != \
                 (prev.cam.pos, prev.cam.right, prev.cam.up, prev.cam.fwd, prev.lens)
    alpha = p.alpha_motion if motion else p.alpha
    vn, vf = pn >= 0, pf >= 0

    def blend(cur, old, has, valid):
        if cur.dim() == 3:
            has, valid = has[..., None], valid[..., None]
        return torch.where(has, torch.where(valid, cur + (old - cur) * alpha, cur), torch.where(valid, old, 0.0))
    accN, accF = blend(near, hA[..., :3], N > 0, vn), blend(far, fB[..., :3], nf > 0, vf)
    accCN, accCF = blend(cN, hC[..., 0], N > 0, vn), blend(cF, fC[..., 1], nf > 0, vf)
    yes = torch.ones_like(on)
    accH = blend(hcur, hA[..., 3], yes, vn)
    huse = hcur if motion else accH
    crt = accF + (accN - accF) * huse[..., None]
    ct = accCF + (accCN - accCF) * huse
    l = _luma(crt)
    mu1, mu2 = blend(l, hC[..., 2], yes, vn), blend(l * l, hC[..., 3], yes, vn)
    var = (mu2 - mu1 * mu1).clamp(min=0) * on
    age = torch.where(vn, hB[..., 3] + 1, 1.0)
    onf = on.double()[..., None]
    out = dict(A=torch.cat([accN, accH[..., None]], 2) * onf, B=torch.cat([accF, age[..., None]], 2) * onf,
               C=torch.stack([accCN, accCF, mu1, mu2], 2) * onf)
    crt, ct, huse = crt * onf, ct * on, huse * on
    out["D"] = vblur = _filter(var, (0.25, 0.5, 0.25), (0.25, 0.5, 0.25))
    # median of the traced neighbours, validity-weighted mips
    nb = [torch.where(v[..., 3:] > 0, v[..., :3], crt) for v in _around(torch.cat([crt, onf], 2))]
    med = torch.stack(nb).median(0).values * onf
    mips = [torch.cat([med, onf], 2)]
    for _ in range(3):
        m = mips[-1]
        m = torch.cat([m, m[-1:]], 0) if m.shape[0] % 2 else m
        m = torch.cat([m, m[:, -1:]], 1) if m.shape[1] % 2 else m
        mips.append((m[0::2, 0::2] + m[0::2, 1::2] + m[1::2, 0::2] + m[1::2, 1::2]) / 4)
    # reconstruction
    recon = torch.zeros((hh, hw, 4), device="cuda", dtype=torch.float64)
    lod = (ct * p.lod_scale).clamp(0, p.lod_max)
    top = 3 if p.lod_max >= 3 else int(p.lod_max)
    tap = torch.stack([torch.where(on, ct, -math.inf), huse], 2)
    for L in range(top + 1):
        at = (on & (lod.floor().long().clamp(max=top) == L)).nonzero(as_tuple=True)
        if not len(at[0]):
            continue
        px, py, c = at[1].double(), at[0].double(), ct[at]
        R, fl = (c / 4).clamp(max=p.r_max), (lod[at] - L)[:, None]
        a, sh, na = torch.zeros((len(c), 4), device="cuda", dtype=torch.float64), 0.0, 0.0
        for ox, oy, frac in _taps():
            sx, sy = px + ox * R, py + oy * R
            v = _at(tap, (sy + 0.5).floor().long(), (sx + 0.5).floor().long())
            ok = (v[:, 0] / 4 >= R * frac).double()
            s = [_bilinear(mips[i], (sx + 0.5) / 2 ** i - 0.5, (sy + 0.5) / 2 ** i - 0.5) for i in (L, min(L + 1, top))]
            a = a + ok[:, None] * torch.lerp(s[0], s[1], fl)
            sh, na = sh + ok * v[:, 1], na + ok
        m = torch.cat([med[at], huse[at][:, None]], 1)
        col = torch.where(a[:, 3:] > 0, a[:, :3] / torch.where(a[:, 3:] > 0, a[:, 3:], 1.0), m[:, :3])
        h = torch.where(na > 0, sh / na.clamp(min=1), m[:, 3])
        b = (vblur[at] * p.var_recon_w).clamp(0, p.b_max)[:, None]
        recon[at] = m + (torch.cat([col, h[:, None]], 1) - m) * b
    # composite at full resolution
    fx = torch.arange(W, device="cuda", dtype=torch.float64)[None, :].expand(H, W) * 0.5 - 0.25
    fy = torch.arange(H, device="cuda", dtype=torch.float64)[:, None].expand(H, W) * 0.5 - 0.25
    up = _bilinear(pp, fx, fy)
    val = _bilinear(torch.cat([recon, ct[..., None], torch.ones_like(onf)], 2) * onf, fx, fy)
    sw = val[..., 5]
    rt = sw > 0
    val = val / torch.where(rt, sw, 1.0)[..., None]
    sharp = (view.coc(depth) <= SQRT2) & (~rt | (val[..., 4] < SQRT2))
    t = sat(val[..., 3] / p.h_edge)
    w = torch.where(depth < d, 1 - up[..., 3], t * t * (3 - 2 * t))[..., None]
    mix = up[..., :3] + (val[..., :3] - up[..., :3]) * w
    res = torch.where(sharp[..., None], colour[..., :3], torch.where(rt[..., None], mix, up[..., :3]))
    return torch.cat([res, torch.ones_like(res[..., :1])], 2), cnt.to(torch.uint8), out


def _inside_around(img):
    """Sum of the eight neighbours inside the image."""
    p = torch.nn.functional.pad(img, (0, 0, 1, 1, 1, 1))
    h, w = img.shape[:2]
    return sum(p[j:j + h, i:i + w] for j in range(3) for i in range(3) if (i, j) != (1, 1))


def exact(case, seed):
    """run's floating outputs in 64 bits, by brute force over all triangles,
    where there are few enough of them; None for the tree (bits, no rounding),
    for large scenes and for a frame's optional stages."""
    kind = case["kind"]
    if kind in ("build", "batch"):
        return None
    px = case.get("width", 0) * case.get("height", 0)
    rays = dict(rays=case.get("rays"), reference=px * case.get("spp", 1), gbuffer=px,
                frame=2 * px + px // 2 * case.get("m", 1))[kind]
    if rays * case["tris"] > MOST_PAIRS:
        return None
    if kind == "frame" and (case["taa"] or case["mask"] == "dilate" or case["polygon"] or px > 1 << 21):
        return None
    scene, cam, lens, pcam, plens, p = _inputs(case, seed)
    world, view = _World(scene), _View(cam, lens)
    if kind == "rays":
        return None, world.hits(*(_t(a) for a in _rays(case, seed, cam, lens)))[1]
    if kind == "gbuffer":
        return _gbuffer64(world, view)
    if kind == "reference":
        n, w, h = case["spp"], cam.width, cam.height
        out = []
        for q in torch.arange(w * h, device="cuda").split(max(1, (1 << 20) // n)):
            o, d = view.lens_rays(q.repeat_interleave(n), torch.arange(n, device="cuda").repeat(len(q)), w, h)
            out.append(world.shade(world.hits(o, d)[0], d)[0].reshape(-1, n, 3).mean(1))
        c = torch.cat(out)
        return torch.cat([c, torch.ones_like(c[:, :1])], 1).reshape(h, w, 4)

    def images(v):
        g = _gbuffer64(world, v)
        # the call's own inputs: 16-bit images and a 32-bit depth
        return [x.half().double() if case["fp16"] and x.dim() == 3 else x.float().double() for x in g]
    before = _View(pcam, plens)
    hist = _frame64(world, before, None, None, images(before), p)[2]
    colour, _, now = _frame64(world, view, _View(pcam, plens, jitter=False), hist, images(view), p)
    flat = torch.cat([now[k].reshape(-1) for k in "ABCD"])
    whole = _history_floats(cam.width, cam.height)
    return dict(colour=colour, mask=None, history=torch.nn.functional.pad(flat, (0, whole - len(flat))))


def _history_floats(w, h):
    """Floats of a history buffer: 13 per half-res pixel, rounded up to 4, then the TAA planes (unused here)."""
    half = (w // 2) * (h // 2)
    return (half * 13 + 3) // 4 * 4 + 8 * w * h + 4 * half
