"""The work that this renderer is used for, as cases that can be timed.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges,
``prepare(case, seed)`` makes what a program holds before the call,
``run(state)`` is one pass through the public entry points, ``work(case)``
the bytes and operations that pass cannot do without, and
``exact(case, seed)`` the same results in 64 bits from plain torch.

A case is a dict of plain values:

  do       frame (forward of camera views), step (forward + backward through
           the autograd Function), rays (forward + adjoint of an explicit ray
           batch with the distortion loss, start cells located first), lens
           (rays of a lens camera generated, located and rendered), load (a
           scene's texels cast, its cells reordered and its records prepared)
  scene    uniform (sites in a cube), shell (a jittered sphere surface in
           uniform background), ellipsoids (20 jittered ellipsoid surfaces,
           seen from a clearing between them); ``sites`` of them
  res      texels per side of a cell's octahedral map
  look     map (one texture), full (surface and view maps), sh (degree 3)
  texels   float32, float16 or bfloat16
  views    pinhole, or mixed (pinhole, fisheye, rolling shutter, thin lens)
  count, width, height   views (mixed: of every kind) and their size
  skip     compositing weight under which a frame skips a texel lookup
  stored   exits per ray that a step's forward keeps for its adjoint
  rays     rays of an explicit batch
"""
from __future__ import annotations

import functools
import math
import os
import subprocess
import sys
import tempfile

import numpy as np
import torch

from paper_2608_17682_amd import autotune, synth, voro
from paper_2608_17682_amd.autograd import render_views

DEV = "cuda:0"
T_STOP = 1e-4
MAX_STEPS = 4096
REACH = {"uniform": 6.0, "shell": 8.0, "ellipsoids": 14.0}   # ray extent
BATCH_VIEWS = 48       # cameras that an explicit ray batch is drawn from
FACES = 15.5           # mean Delaunay degree of a cell


# ------------------------------------------------------------------ cases

def _case(name, do, scene, sites, res=8, look="map", texels="float32", views="pinhole", count=1,
          width=0, height=0, skip=0.0, stored=0, rays=0):
    c = {"do": do, "scene": scene, "sites": sites, "res": res, "look": look, "texels": texels,
         "views": views, "count": count, "width": width, "height": height, "skip": skip,
         "stored": stored, "rays": rays}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest calls: a thumbnail of a toy scene, where launches and host time count
        _case("frame_uniform512", "frame", "uniform", 512, res=4, width=64, height=64),
        # one training step at the same size
        _case("step_uniform512", "step", "uniform", 512, res=4, width=64, height=64, stored=256),
        # a viewer's frame of an object-sized scene
        _case("frame_shell100k", "frame", "shell", 100_000, width=800, height=800),
        # the viewer's fast settings: the two-map model in binary16 with the cell skip
        _case("frame_shell100k_full", "frame", "shell", 100_000, look="full", texels="float16",
              width=1280, height=840, skip=1e-3),
        # the spherical-harmonic comparison model
        _case("frame_shell100k_sh", "frame", "shell", 100_000, look="sh", width=800, height=800),
        # training on whole views
        _case("step_shell100k", "step", "shell", 100_000, width=800, height=800, stored=256),
        # training of the two-map model
        _case("step_shell100k_full", "step", "shell", 100_000, look="full", width=800,
              height=800, stored=256),
        # training on a batch of random pixels of many views, with the distortion
        # loss: rays of a wave have nothing to do with each other; a ragged size
        _case("rays_shell100k", "rays", "shell", 100_000, stored=128, rays=131_071),
        # depth of field through the explicit-ray entry points, bfloat16 texels, odd size
        _case("lens_shell100k", "lens", "shell", 100_000, texels="bfloat16", width=323,
              height=241),
        # training of a full-sized scene from inside it
        _case("step_ellipsoids2M", "step", "ellipsoids", 2_000_000, width=1280, height=840,
              stored=256),
        # the largest: 4M sites and 8 mixed views a launch, forward + backward
        _case("step_shell4M_views", "step", "shell", 4_000_000, texels="float16", views="mixed",
              count=2, width=1280, height=840, stored=256),
        # a scene on its way into a viewer
        _case("load_ellipsoids2M", "load", "ellipsoids", 2_000_000, texels="float16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["frame", "frame", "step", "step", "rays", "lens", "load"])
    sites = _log(rng, 512, 1_200_000)
    scene = "uniform" if sites < 5000 else rng.choice(["shell", "shell", "ellipsoids"])
    res = rng.choice([4, 8, 8, rng.randint(3, 10)])
    look = rng.choice(["map", "map", "full"] + (["sh"] if do in ("frame", "lens") else []))
    texels = rng.choice(["float32", "float32", "float16", "bfloat16"])
    if do == "load" and texels == "float32":
        texels = "float16"
    if do in ("rays", "load"):
        look = "map"
    if do == "load":
        res = rng.choice([4, 8])   # as scenes are stored
    views = rng.choice(["pinhole", "pinhole", "mixed"]) if do in ("frame", "step") else "pinhole"
    px = _log(rng, 2_000, 900_000 if views == "pinhole" else 200_000)
    if do == "lens":
        px = min(px, 250_000)
    width = max(8, int(math.sqrt(px * rng.uniform(0.8, 1.8))))
    height = max(8, px // width)
    return _case("", do, scene, sites, res, look, texels, views,
                 rng.randint(1, 2) if views == "pinhole" else 1,
                 width if do not in ("rays", "load") else 0,
                 height if do not in ("rays", "load") else 0,
                 rng.choice([0.0, 0.0, 1e-3]) if do == "frame" else 0.0,
                 rng.choice([0, 64, 256]) if do in ("step", "rays") else 0,
                 _log(rng, 1_000, 300_000) if do == "rays" else 0)


# ------------------------------------------------------------------- scenes

_BUILD = """
import sys
sys.path.insert(0, sys.argv[1])
from perf import cases
cases._save_geometry(sys.argv[2], int(sys.argv[3]), sys.argv[4])
"""


def _build_geometry(kind, n):
    """Sites, surface-or-background densities and adjacency of a scene, cells in
    Morton order (as a loaded scene holds them), and a point with a view."""
    eye = target = np.zeros(3)
    if kind == "uniform":
        s = synth.scene_uniform(n, 2, seed=1)
    elif kind == "shell":
        s = synth.scene_shell(n, 2, seed=2)
    else:
        back = max(20, n // 10)
        per = (n - back) // 20
        s, ells, rng = synth.scene_ellipsoids(per * 20, n - per * 20, tex_res=2)
        c2w = synth.interior_camera(ells, rng).c2w
        eye, target = c2w[:, 3], c2w[:, 3] + c2w[:, 2]
    lo, hi = s.sites.min(0), s.sites.max(0)
    q = np.clip((s.sites - lo) / np.maximum(hi - lo, 1e-30) * 1024, 0, 1023).astype(np.int64)
    code = np.zeros(len(q), np.int64)
    for b in range(10):
        for a in range(3):
            code |= ((q[:, a] >> b) & 1) << (3 * b + 2 - a)
    given = [torch.from_numpy(v) for v in (s.sites, s.density, s.nbr_off, s.nbr_idx)]
    geo = _reordered(*given, torch.from_numpy(np.argsort(code, kind="stable")))
    return dict({k: v.numpy() for k, v in geo.items()}, eye=eye, target=target)


def _reordered(sites, density, off, idx, perm):
    """The scene (tensors) with cell k = the given scene's cell perm[k]."""
    inv = torch.empty_like(perm)
    inv[perm] = torch.arange(len(perm), device=perm.device)
    start = off.long()
    deg = (start[1:] - start[:-1])[perm]
    new = torch.cat([deg.new_zeros(1), torch.cumsum(deg, 0)])
    at = torch.arange(len(idx), device=perm.device)
    at = at + torch.repeat_interleave(start[:-1][perm] - new[:-1], deg)
    return {"sites": sites[perm], "density": density[perm], "off": new.int(),
            "idx": inv[idx[at].long()].int()}


def _save_geometry(kind, n, path):
    np.savez(path, **_build_geometry(kind, n))


@functools.lru_cache(maxsize=4)
def _geometry(kind, n):
    """The geometry of a size is built once; big ones in a child process, which
    forks workers, and kept on disk for the next program."""
    if n <= 5000:
        return _build_geometry(kind, n)
    folder = os.path.join(tempfile.gettempdir(), f"voro_cases_{os.getuid()}")
    os.makedirs(folder, exist_ok=True)
    path = os.path.join(folder, f"{kind}_{n}.npz")
    if not os.path.exists(path):
        part = f"{path[:-4]}.{os.getpid()}.npz"
        subprocess.run([sys.executable, "-c", _BUILD, os.getcwd(), kind, str(n), part], check=True)
        os.replace(part, path)
    with np.load(path, allow_pickle=False) as z:
        return {k: z[k] for k in z.files}


def _turn(rng):
    """A random rotation."""
    q, r = np.linalg.qr(rng.normal(size=(3, 3)))
    q = q * np.sign(np.diag(r))
    return q if np.linalg.det(q) > 0 else -q


def _inputs(case, seed):
    """Everything the seed decides: the scene turned by a random rotation (its
    adjacency turns with it), densities, texels, cameras, upstream gradients."""
    rng = np.random.default_rng([seed, case["sites"]])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(rng.integers(1 << 62)))
    geo = _geometry(case["scene"], case["sites"])
    turn = _turn(rng)
    n, res = len(geo["sites"]), case["res"]
    x = {"n": n, "sites": torch.from_numpy((geo["sites"] @ turn.T).astype(np.float32)).to(DEV)}
    spread = torch.randn(n, generator=gen, device=DEV)
    x["density"] = torch.from_numpy(geo["density"]).to(DEV) * torch.exp(0.2 * spread)
    x["off"], x["idx"] = (torch.from_numpy(geo[k]).to(DEV) for k in ("off", "idx"))
    dtype = getattr(torch, case["texels"])
    if case["look"] == "sh":
        # a base colour and higher orders that fall off
        k = torch.randn((n, 16, 3), generator=gen, device=DEV)
        fall = [0.15 / 2 ** int(math.isqrt(i)) for i in range(16)]
        k *= torch.tensor(fall, device=DEV)[None, :, None]
        k[:, 0] = (0.2 + 0.6 * torch.rand((n, 3), generator=gen, device=DEV)) * 2 * math.sqrt(math.pi)
        x["texels"] = k.reshape(n, 48).to(dtype)
    elif case["look"] == "full":
        t = torch.randn((n, 2, res, res, 4), generator=gen, device=DEV)
        t *= torch.tensor([1.5, 0.5], device=DEV)[None, :, None, None, None]
        t[..., 3] = 0.0
        x["texels"] = t.to(dtype)
    else:
        t = torch.rand((n, res, res, 4), generator=gen, device=DEV)
        t[..., 3] = 0.0
        x["texels"] = t if case["do"] == "load" else t.to(dtype)
    x["cams"] = _cameras(case, rng, geo, turn)
    pixels = sum(c.n_pixels for c in x["cams"])
    if case["do"] == "rays":
        x.update(_batch(case, gen, x["cams"]))
        pixels = case["rays"]
    for name, shape in (("g_rgb", (pixels, 3)), ("g_T", (pixels,)), ("g_dist", (pixels,))):
        x[name] = torch.randn(shape, generator=gen, device=DEV)
    if case["do"] == "load":
        x["shuffle"] = torch.randperm(n, generator=gen, device=DEV)
    return x


def _cameras(case, rng, geo, turn):
    reach = REACH[case["scene"]]

    def pose(k, of):
        if case["scene"] == "ellipsoids":
            eye, at = geo["eye"], geo["target"] - geo["eye"]
            at = at + rng.normal(scale=0.15, size=3)
        else:
            a = 2.0 * math.pi * (k + rng.uniform(0, 1)) / of
            eye = 3.0 * np.array([math.sin(a), rng.uniform(-0.3, 0.3), -math.cos(a)])
            at = -eye
        return synth.look_at(turn @ eye, turn @ (eye + at), turn @ np.array([0.0, 1.0, 0.0]))

    w, h, fov = case["width"], case["height"], math.radians(60.0)
    if case["do"] == "load":
        return []
    if case["do"] == "rays":
        return [synth.Camera(synth.PINHOLE, 800, 800, pose(k, BATCH_VIEWS), fov, reach)
                for k in range(BATCH_VIEWS)]
    if case["do"] == "lens":
        return [synth.Camera(synth.THIN_LENS, w, h, pose(0, 1), fov, reach, lens_radius=0.05,
                             focus_dist=3.0, spp=4)]
    out = []
    kinds = ("pinhole",) if case["views"] == "pinhole" else ("pinhole", "fisheye", "rolling", "lens")
    for m, kind in enumerate(kinds):
        for k in range(case["count"]):
            c = pose(m * case["count"] + k, len(kinds) * case["count"])
            if kind == "pinhole":
                out.append(synth.Camera(synth.PINHOLE, w, h, c, fov, reach))
            elif kind == "fisheye":   # a square image of about the same area
                s = max(2, int(round(math.sqrt(w * h))) // 8 * 8)
                out.append(synth.Camera(synth.FISHEYE, s, s, c, math.pi, reach))
            elif kind == "rolling":
                out.append(synth.Camera(synth.ROLLING_SHUTTER, max(2, w * 3 // 4),
                                        max(2, h * 9 // 14), c, fov, reach,
                                        rs_delta=tuple(float(v) for v in 0.1 * c[:, 0])))
            else:
                out.append(synth.Camera(synth.THIN_LENS, max(2, w // 2), max(2, h * 4 // 7), c,
                                        fov, reach, lens_radius=0.05, focus_dist=3.0, spp=4))
    return out


def _batch(case, gen, cams):
    """Random pixels of the views: unit directions, the view of each ray."""
    R = case["rays"]
    view = torch.randint(0, len(cams), (R,), generator=gen, device=DEV)
    px = torch.rand((R, 2), generator=gen, device=DEV, dtype=torch.float64)
    m = torch.tensor(np.stack([c.c2w for c in cams]), device=DEV)
    u = (2.0 * px - 1.0) * math.tan(0.5 * cams[0].fov)
    d = torch.cat([u, torch.ones_like(u[:, :1])], 1)
    d = (m[view][:, :, :3] @ d[:, :, None])[..., 0]
    d = d / d.norm(dim=1, keepdim=True)
    centres = m[:, :, 3].float().contiguous()
    return {"o": centres[view].contiguous(), "d": d.float().contiguous(),
            "tmax": torch.full((R,), cams[0].tmax, device=DEV), "centres": centres, "view": view}


# ---------------------------------------------------------------------- runs

def prepare(case, seed):
    x = _inputs(case, seed)
    s = {"case": dict(case), "x": x}
    arrays = [x["sites"], x["density"], x["off"], x["idx"], x["texels"]]
    if case["do"] == "load":
        # the cells as they come out of training: in no order
        geo = _reordered(*arrays[:4], x["shuffle"])
        s["arrays"] = [geo[k] for k in ("sites", "density", "off", "idx")] + arrays[4:]
        return s
    ds = voro.DeviceScene(*arrays)
    s["ds"] = ds
    s["cams"] = [voro.camera_of(c) for c in x["cams"]]
    look = {"map": 0, "full": 1, "sh": 2}[case["look"]]
    s["fwd"] = autotune.params_for(ds, x["cams"], "fwd")
    s["bwd"] = autotune.params_for(ds, x["cams"], "bwd")
    for p in (s["fwd"], s["bwd"]):
        p.appearance = look
    s["fwd"].skip_w = case["skip"]
    if case["do"] == "step":
        s["leaves"] = [t.requires_grad_(True) for t in (x["sites"], x["density"], x["texels"])]
    else:
        voro.voro_prepare(ds)
    if case["do"] in ("rays", "lens"):
        s["params"] = voro.default_params(appearance=look)
    if case["do"] == "lens":
        s["centres"] = torch.tensor([[c.c2w[3], c.c2w[7], c.c2w[11]] for c in s["cams"]],
                                    dtype=torch.float32, device=DEV)
    return s


def run(s):
    return _RUN[s["case"]["do"]](s)


def _run_frame(s):
    rgb, T, _ = voro.voro_render_views_fwd(s["ds"], s["cams"], s["fwd"])
    return {"rgb": rgb, "T": T}


def _run_step(s):
    x, case = s["x"], s["case"]
    rgb, T = render_views(*s["leaves"], x["off"], x["idx"], s["cams"], s["fwd"], s["bwd"],
                          stored_exits=case["stored"])
    g = torch.autograd.grad((rgb, T), s["leaves"], (x["g_rgb"], x["g_T"]))
    return {"rgb": rgb, "T": T, "g_sites": g[0], "g_density": g[1], "g_texels": g[2]}


def _run_rays(s):
    """A training iteration on a ray batch: the sites have moved, so the records
    are prepared and the cells of the camera centres looked up again."""
    x, ds, p, stored = s["x"], s["ds"], s["params"], s["case"]["stored"]
    voro.voro_prepare(ds)
    start = voro.voro_locate_origins(ds, x["centres"])[x["view"]]
    R = s["case"]["rays"]
    dist = torch.empty((R, 3), device=DEV)
    trace = torch.empty((stored, R, 2), dtype=torch.int32, device=DEV) if stored else None
    rgb, T = voro.voro_render_fwd(ds, x["o"], x["d"], x["tmax"], start, p, dist=dist, trace=trace)
    gs, gd, gt = voro.voro_render_bwd(ds, x["o"], x["d"], x["tmax"], start, rgb, T, x["g_rgb"],
                                      x["g_T"], p, dist=dist, g_dist=x["g_dist"], trace=trace)
    return {"rgb": rgb, "T": T, "dist": dist[:, 0], "start": start, "g_sites": gs,
            "g_density": gd, "g_texels": gt}


def _run_lens(s):
    ds = s["ds"]
    o, d, tmax = voro.voro_gen_rays(s["cams"], DEV)
    centre = voro.voro_locate_origins(ds, s["centres"])
    start = voro.voro_locate_origins(ds, o, hint=centre.expand(len(o)).contiguous())
    rgb, T = voro.voro_render_fwd(ds, o, d, tmax, start, s["params"])
    return {"rgb": rgb, "T": T, "start": start}


def _run_load(s):
    sites, density, off, idx, tex = s["arrays"]
    half = voro.voro_cast_texels(tex, s["case"]["texels"])
    ds, perm, inv = voro.voro_morton_reorder(voro.DeviceScene(sites, density, off, idx, half))
    voro.voro_prepare(ds)
    return {"sites": ds.sites, "density": ds.density, "off": ds.nbr_off, "idx": ds.nbr_idx,
            "texels": ds.texels, "perm": perm, "inv": inv}


_RUN = {"frame": _run_frame, "step": _run_step, "rays": _run_rays, "lens": _run_lens,
        "load": _run_load}


# ---------------------------------------------------------------------- work

def _steps(case):
    """Mean cells along a ray: about n^(1/3), with the surfaces' share."""
    n = case["sites"]
    if case["scene"] == "uniform":
        return 1.4 * n ** (1 / 3)
    return (45.5 * (n / 1e5) ** 0.31 if case["scene"] == "shell"
            else 59.9 * (n / 2e6) ** 0.31)


def _image(case):
    """Rays and pixels of the views."""
    w, h, k = case["width"], case["height"], case["count"]
    if case["do"] == "rays":
        return case["rays"], case["rays"]
    if case["do"] == "lens":
        return 4 * w * h, 4 * w * h
    if case["views"] == "pinhole":
        return w * h * k, w * h * k
    lens = max(2, w // 2) * max(2, h * 4 // 7)
    rolling = max(2, w * 3 // 4) * max(2, h * 9 // 14)
    fish = max(2, int(round(math.sqrt(w * h))) // 8 * 8) ** 2
    return (k * (w * h + fish + rolling + 4 * lens), k * (w * h + fish + rolling + lens))


def work(case):
    n = case["sites"]
    size = 4 if case["texels"] == "float32" else 2
    values = 48 if case["look"] == "sh" else 4 * case["res"] ** 2 * (2 if case["look"] == "full" else 1)
    cells, tex = n * (12 + 4 + 4 + 4 * FACES), n * values * size
    if case["do"] == "load":   # scene in and out, the casted texels, records written
        return {"bytes": 2 * cells + n * values * 4 + tex + 8 * n + n * (32 + 16 * FACES),
                "flops": n * 20.0 * FACES}
    rays, pixels = _image(case)
    steps = rays * _steps(case)
    # a walk needs no more of the scene than it visits
    step_bytes = 24 + 16 * FACES + {"sh": 48 * size, "full": 32 * size}.get(case["look"], 16 * size)
    bytes_ = min(cells + tex, steps * step_bytes) + 16 * pixels
    flops = steps * (14 * FACES + 60)
    if case["do"] == "step" or case["do"] == "rays":   # gradients out, upstream in
        bytes_ += n * 16 + n * values * (size if case["do"] == "step" else 4) + 32 * pixels
        flops += steps * 120
    return {"bytes": float(bytes_), "flops": float(flops)}


# ------------------------------------------------------- the same in 64 bits

def exact(case, seed):
    if case["do"] == "load":
        return None   # copies, whole numbers and one rounding
    rays, _ = _image(case)
    if rays * _steps(case) > 1.2e8:
        return None   # minutes in 64 bits
    x = _inputs(case, seed)
    f = {k: x[k].double() for k in ("sites", "density", "texels", "g_rgb", "g_T", "g_dist")}
    off, idx = x["off"].long(), x["idx"].long()
    if case["do"] == "rays":
        cell = _nearest(f["sites"], x["centres"].double())
        o, d, tmax, start = x["o"].double(), x["d"].double(), x["tmax"].double(), cell[x["view"]]
        pixel, share = torch.arange(len(o), device=DEV), 1.0
    else:
        o, d, tmax, start, pixel, share = _camera_rays(x["cams"], f["sites"], off, idx)
    if case["do"] == "lens":   # every sample is a ray of its own
        pixel, share = torch.arange(len(o), device=DEV), 1.0
    P = int(pixel.max()) + 1
    share = share if torch.is_tensor(share) else torch.full((len(o),), share, device=DEV,
                                                            dtype=torch.float64)
    out = {"rgb": torch.zeros((P, 3), device=DEV, dtype=torch.float64),
           "T": torch.zeros(P, device=DEV, dtype=torch.float64)}
    grads = case["do"] in ("step", "rays")
    if grads:
        out.update(g_sites=torch.zeros_like(f["sites"]), g_density=torch.zeros_like(f["density"]),
                   g_texels=torch.zeros_like(f["texels"]))
    if case["do"] == "rays":
        out["dist"] = torch.zeros(P, device=DEV, dtype=torch.float64)
    per = max(4096, int(6e6 / _steps(case)))
    for a in range(0, len(o), per):
        k = slice(a, a + per)
        _trace64(case, f, off, idx, o[k], d[k], tmax[k], start[k], pixel[k], share[k], out, grads)
    if case["do"] in ("rays", "lens"):
        out["start"] = None
    return out


def _nearest(sites, points):
    out = []
    for p in points:
        out.append(((sites - p) ** 2).sum(1).argmin())
    return torch.stack(out)


def _ragged(off, cur):
    """Rows of the cells cur, end to end: (owner of each entry, its place)."""
    deg = off[cur + 1] - off[cur]
    owner = torch.repeat_interleave(torch.arange(len(cur), device=DEV), deg)
    first = torch.cumsum(deg, 0) - deg
    return owner, torch.arange(len(owner), device=DEV) - first[owner] + off[cur][owner]


def _walk_to(sites, off, idx, points, start):
    """Nearest sites, by steps to the closest neighbour while one is closer."""
    cur, todo = start.clone(), torch.arange(len(points), device=DEV)
    while len(todo):
        own, at = _ragged(off, cur[todo])
        j = idx[at]
        d2 = ((sites[j] - points[todo][own]) ** 2).sum(1)
        best = torch.full((len(todo),), math.inf, device=DEV, dtype=torch.float64)
        best.scatter_reduce_(0, own, d2, "amin")
        pick = torch.full((len(todo),), len(sites), device=DEV, dtype=torch.int64)
        pick.scatter_reduce_(0, own, torch.where(d2 == best[own], j, len(sites)), "amin")
        here = ((sites[cur[todo]] - points[todo]) ** 2).sum(1)
        go = best < here
        cur[todo[go]] = pick[go]
        todo = todo[go]
    return cur


def _camera_rays(cams, sites, off, idx):
    """Rays of the views in order, pixels row-major, then samples."""
    parts, first = [], 0
    for c in cams:
        M = torch.tensor(np.asarray(c.c2w, np.float32).astype(np.float64), device=DEV)
        fov, W, H, spp = float(np.float32(c.fov)), c.width, c.height, c.spp
        i = torch.arange(W * H * spp, device=DEV)
        pix, s = i // spp, i % spp
        u = (pix % W).double() + 0.5 - 0.5 * W
        v = torch.div(pix, W, rounding_mode="floor").double() + 0.5 - 0.5 * H
        o = M[:, 3].expand(len(i), 3)
        tmax = torch.full((len(i),), float(np.float32(c.tmax)), device=DEV, dtype=torch.float64)
        one = torch.ones_like(u)
        if c.model == synth.FISHEYE:
            r = torch.sqrt(u * u + v * v)
            th = r / ((0.5 * W) / (0.5 * fov))
            q = torch.stack([torch.sin(th) * u / r.clamp(min=1e-300),
                             torch.sin(th) * v / r.clamp(min=1e-300), torch.cos(th)], 1)
            tmax = torch.where(r * r <= 0.25 * W * W, tmax, 0.0)
        else:
            focal = (0.5 * W) / math.tan(0.5 * fov)
            q = torch.stack([u / focal, v / focal, one], 1)
            if c.model == synth.ROLLING_SHUTTER:
                row = torch.div(pix, W, rounding_mode="floor").double() / (H - 1)
                delta = torch.tensor(np.asarray(c.rs_delta, np.float32).astype(np.float64), device=DEV)
                o = o + row[:, None] * delta
            if c.model == synth.THIN_LENS:
                g = int(round(math.sqrt(spp)))
                a = 2.0 * ((s % g).double() + 0.5) / g - 1.0
                b = 2.0 * (torch.div(s, g, rounding_mode="floor").double() + 0.5) / g - 1.0
                wide = a.abs() > b.abs()
                r = torch.where(wide, a, b)
                phi = torch.where(wide, 0.25 * math.pi * b / torch.where(wide, a, 1.0),
                                  0.5 * math.pi - 0.25 * math.pi * a / torch.where(b != 0, b, 1.0))
                centre = (a == 0) & (b == 0)
                rad, foc = float(np.float32(c.lens_radius)), float(np.float32(c.focus_dist))
                lx = torch.where(centre, 0.0, r * torch.cos(phi)) * rad
                ly = torch.where(centre, 0.0, r * torch.sin(phi)) * rad
                q = torch.stack([foc * q[:, 0] - lx, foc * q[:, 1] - ly, foc * one], 1)
                o = o + lx[:, None] * M[:, 0] + ly[:, None] * M[:, 1]
        d = q @ M[:, :3].T
        d = d / d.norm(dim=1, keepdim=True)
        at = _nearest(sites, M[None, :, 3]).expand(len(i))
        if c.model in (synth.ROLLING_SHUTTER, synth.THIN_LENS):
            at = _walk_to(sites, off, idx, o, at)
        parts.append((o, d, tmax, at, first + pix, torch.full_like(u, 1.0 / spp)))
        first += W * H
    return tuple(torch.cat(p) for p in zip(*parts))


def _sequence(case, f, off, idx, o, d, tmax, start):
    """The walk: for every visited cell its ray, itself, the next cell (-1: none)
    and the visit whose exit last advanced the ray (-1: none), ray by ray."""
    P, N = f["sites"], len(f["sites"])
    live = torch.nonzero(tmax > 0)[:, 0]
    cur, t_in, T = start.clone(), torch.zeros_like(tmax), torch.ones_like(tmax)
    last = torch.full((len(o),), -1, device=DEV, dtype=torch.int64)
    rows = []
    for k in range(MAX_STEPS):
        if not len(live):
            break
        c = cur[live]
        own, at = _ragged(off, c)
        j = idx[at]
        nv = P[j] - P[c][own]
        b = (nv * d[live][own]).sum(1)
        num = (nv * (0.5 * (P[j] + P[c][own]) - o[live][own])).sum(1)
        t = torch.where(b > 0, num / b, math.inf)
        exit_t = torch.full((len(live),), math.inf, device=DEV, dtype=torch.float64)
        exit_t.scatter_reduce_(0, own, t, "amin")
        nxt = torch.full((len(live),), N, device=DEV, dtype=torch.int64)
        nxt.scatter_reduce_(0, own, torch.where((t == exit_t[own]) & torch.isfinite(t), j, N), "amin")
        nxt = torch.where(nxt == N, -1, nxt)
        rows.append((live, torch.full_like(live, k), c, nxt, last[live]))
        t_out = torch.minimum(exit_t, tmax[live])
        T[live] *= torch.exp(-f["density"][c] * (t_out - t_in[live]).clamp(min=0))
        go = (T[live] >= T_STOP) & (exit_t < tmax[live]) & (nxt >= 0)
        further = t_out > t_in[live]
        last[live] = torch.where(further, k, last[live])
        t_in[live] = torch.maximum(t_in[live], t_out)
        cur[live] = torch.where(go, nxt, c)
        live = live[go]
    ray, k, cell, nxt, last = (torch.cat(r) for r in zip(*rows))
    order = torch.argsort(ray * MAX_STEPS + k)
    ray, k, cell, nxt, last = (v[order] for v in (ray, k, cell, nxt, last))
    first = torch.full((len(o),), len(ray), device=DEV, dtype=torch.int64)
    first.scatter_reduce_(0, ray, torch.arange(len(ray), device=DEV), "amin")
    return ray, k, cell, nxt, torch.where(last >= 0, first[ray] + last, -1), first


def _taps(d, R):
    """Octahedral lookup at directions d: base texel and the four weights."""
    q = d / d.abs().sum(1, keepdim=True)
    sx, sy = (torch.where(q[:, i] >= 0, 1.0, -1.0) for i in (0, 1))
    up = q[:, 2] >= 0
    u = torch.where(up, q[:, 0], (1 - q[:, 1].abs()) * sx)
    v = torch.where(up, q[:, 1], (1 - q[:, 0].abs()) * sy)
    x, y = (u + 1) * 0.5 * (R - 1), (v + 1) * 0.5 * (R - 1)
    cx, cy = (z.detach().floor().clamp(0, R - 2) for z in (x, y))
    fx, fy = x - cx, y - cy
    w = torch.stack([(1 - fx) * (1 - fy), fx * (1 - fy), (1 - fx) * fy, fx * fy], 1)
    return (cy * R + cx).long(), w


def _harmonics(d):
    """Real orthonormal spherical harmonics up to degree 3, no Condon-Shortley phase."""
    x, y, z = d.unbind(1)
    pi = math.pi
    a, b = math.sqrt(3 / (4 * pi)), math.sqrt(15 / pi) / 2
    c, e = math.sqrt(35 / (2 * pi)) / 4, math.sqrt(21 / (2 * pi)) / 4
    return torch.stack([
        torch.full_like(x, 0.5 / math.sqrt(pi)), a * y, a * z, a * x,
        b * x * y, b * y * z, math.sqrt(5 / pi) / 4 * (3 * z * z - 1), b * x * z,
        b / 2 * (x * x - y * y), c * y * (3 * x * x - y * y), math.sqrt(105 / pi) / 2 * x * y * z,
        e * y * (5 * z * z - 1), math.sqrt(7 / pi) / 4 * z * (5 * z * z - 3),
        e * x * (5 * z * z - 1), math.sqrt(105 / pi) / 4 * z * (x * x - y * y),
        c * x * (x * x - 3 * y * y)], 1)


def _trace64(case, f, off, idx, o, d, tmax, start, pixel, share, out, grads):
    """Renders some rays in 64 bits into `out`: the cells along them first, then
    their colours as one expression of the visited cells, which autograd
    differentiates."""
    ray, k, cell, nxt, entry, first = _sequence(case, f, off, idx, o, d, tmax, start)
    n_rays = len(o)
    pa, pb = f["sites"][cell], f["sites"][nxt.clamp(min=0)]
    sigma = f["density"][cell]
    leaves = [v.requires_grad_(grads) for v in (pa, pb, sigma)]
    dr, orr = d[ray], o[ray]
    nv = pb - pa
    beta = torch.where(nxt >= 0, (nv * dr).sum(1), 1.0)
    t_ex = (nv * (0.5 * (pa + pb) - orr)).sum(1) / beta
    t_ex = torch.where(nxt >= 0, t_ex, math.inf)
    t_out = torch.where(t_ex < tmax[ray], t_ex, tmax[ray])
    t_in = torch.where(entry >= 0, t_out[entry.clamp(min=0)], 0.0)
    tau = sigma * (t_out - t_in).clamp(min=0)
    total = torch.cumsum(tau, 0)
    before = torch.cat([total.new_zeros(1), total])[first.clamp(max=len(ray))][ray]
    T = torch.exp(-(total - tau - before))
    w = T * -torch.expm1(-tau)
    # colours
    R, maps = case["res"], 2 if case["look"] == "full" else 1
    taps = []

    def lookup(at, weight):
        flat = f["texels"].view(-1, 4)[:, :3]
        rows = (at[:, None] + torch.tensor([0, 1, R, R + 1], device=DEV))
        t = flat[rows].requires_grad_(grads)
        taps.append((rows, t))
        return (t * weight[..., None]).sum(1)

    if case["look"] == "sh":
        colour = (f["texels"].view(-1, 16, 3)[cell] * _harmonics(d)[ray][..., None]).sum(1)
    elif case["look"] == "full":
        th = torch.where(k > 0, t_in, t_out)
        base, wt = _taps(orr + th[:, None] * dr - pa, R)
        logit = lookup(2 * cell * R * R + base, wt)
        base, wt = _taps(-d, R)
        colour = torch.sigmoid(logit + lookup((2 * cell + 1) * R * R + base[ray], wt[ray]))
    else:
        base, wt = _taps(d, R)
        colour = lookup(cell * R * R + base[ray], wt[ray])
    kept = torch.where(w >= float(np.float32(case["skip"])), w, 0.0)
    rgb = torch.zeros((n_rays, 3), device=DEV, dtype=torch.float64).index_add(0, ray, kept[:, None] * colour)
    Tf = torch.exp(-torch.zeros(n_rays, device=DEV, dtype=torch.float64).index_add(0, ray, tau))
    out["rgb"].index_add_(0, pixel, rgb.detach() * share[:, None])
    out["T"].index_add_(0, pixel, Tf.detach() * share)
    if not grads:
        return
    loss = (rgb * f["g_rgb"][pixel] * share[:, None]).sum() + (Tf * f["g_T"][pixel] * share).sum()
    if case["do"] == "rays":
        s0, s1 = t_in / (1 + t_in), t_out / (1 + t_out)
        s1 = torch.maximum(s0, s1)
        mid = 0.5 * (s0 + s1)

        def earlier(v):
            c = torch.cumsum(v, 0)
            return c - v - torch.cat([c.new_zeros(1), c])[first.clamp(max=len(ray))][ray]

        part = 2 * w * (mid * earlier(w) - earlier(w * mid)) + w * w * (s1 - s0) / 3
        dist = torch.zeros(n_rays, device=DEV, dtype=torch.float64).index_add(0, ray, part)
        out["dist"].index_add_(0, pixel, dist.detach())
        loss = loss + (dist * f["g_dist"][pixel]).sum()
    got = torch.autograd.grad(loss, leaves + [t for _, t in taps])
    out["g_sites"].index_add_(0, cell, got[0])
    out["g_sites"].index_add_(0, nxt.clamp(min=0), torch.where((nxt >= 0)[:, None], got[1], 0.0))
    out["g_density"].index_add_(0, cell, got[2])
    g = out["g_texels"].view(-1, 4)
    for (rows, _), grad in zip(taps, got[3:]):
        v = torch.cat([grad, torch.zeros_like(grad[..., :1])], -1)
        g.index_add_(0, rows.reshape(-1), v.reshape(-1, 4))
