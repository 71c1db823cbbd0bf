"""Forward kernels with one lane per ray, which stage the edge rows of a wave's
cells, against two lanes per ray, which stage nothing, bit by bit: rows and waves
around what can be staged, cells without faces, malformed rows, every appearance
model, texel type and schedule, and the ray count from which the kernels are held
to a fifth wave per SIMD.  (Small launches take more lanes unless they ask.)"""
import numpy as np
import pytest
import torch

from paper_2608_17682_amd import synth, voro

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    voro.lib()
    return torch.device("cuda:0")


def to_dev(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


@pytest.mark.parametrize("rays", [262_144, 262_145])
@pytest.mark.parametrize("look", ["map", "full"])
def test_ray_counts_around_the_fifth_wave(dev, rays, look):
    print(f"[gpu-case] one lane, {rays} rays, {look}", flush=True)
    sc = synth.scene_uniform(512, 4, seed=71)
    tex = synth.full_texels(sc.n, 4, seed=72) if look == "full" else sc.texels
    ds = voro.DeviceScene(to_dev(sc.sites, dev), to_dev(sc.density, dev), to_dev(sc.nbr_off, dev),
                          to_dev(sc.nbr_idx, dev), to_dev(tex, dev))
    voro.voro_prepare(ds)
    gen = torch.Generator(device=dev).manual_seed(73)
    o = torch.rand((rays, 3), generator=gen, device=dev) * 1.8 - 0.9
    d = torch.nn.functional.normalize(torch.randn((rays, 3), generator=gen, device=dev), dim=1)
    # half of the waves in bundles (staged rows), half scattered (gathered ones)
    d[: rays // 128 * 64] = d[: rays // 128].repeat_interleave(64, 0)
    o[: rays // 128 * 64] = o[: rays // 128].repeat_interleave(64, 0)
    start = voro.voro_locate_origins(ds, o)
    tm = torch.full((rays,), 1.5, device=dev)
    out = []
    for lanes in (1, 2):
        k = torch.empty(rays, dtype=torch.int32, device=dev)
        p = voro.default_params(lanes_per_ray=lanes, appearance=1 if look == "full" else 0)
        out.append((*voro.voro_render_fwd(ds, o, d, tm, start, p, nsteps=k), k))
    for a, b in zip(*out):
        assert torch.equal(a, b)
    assert int(out[0][2].max()) > 3


def upload(dev, sites, density, tex, off, idx):
    ds = voro.DeviceScene(to_dev(np.asarray(sites, np.float32), dev),
                          to_dev(np.asarray(density, np.float32), dev),
                          to_dev(np.asarray(off, np.int32), dev),
                          to_dev(np.asarray(idx, np.int32), dev), to_dev(tex, dev))
    voro.voro_prepare(ds)
    return ds


def unit(d):
    return (d / np.linalg.norm(d, axis=-1, keepdims=True)).astype(np.float32)


def walks(dev, ds, o, d, start, tmax=3.0, **kw):
    """Steps per ray, the outputs of one and of two lanes having been found equal."""
    O, D, S = to_dev(o.astype(np.float32), dev), to_dev(d, dev), to_dev(start.astype(np.int32), dev)
    TM = torch.full((len(o),), tmax, device=dev)
    out = []
    for lanes in (1, 2):
        p = voro.default_params(lanes_per_ray=lanes, max_record=32, **kw)
        k = torch.empty(len(o), dtype=torch.int32, device=dev)
        cells = torch.empty((len(o), 32), dtype=torch.int32, device=dev)
        dist = torch.empty((len(o), 3), device=dev)
        st = torch.zeros(voro.STAT_COUNT, dtype=torch.int64, device=dev)
        rgb, T = voro.voro_render_fwd(ds, O, D, TM, S, p, nsteps=k, cells=cells, dist=dist, stats=st)
        assert torch.isfinite(rgb).all() and torch.isfinite(T).all()
        out.append((rgb, T, k, cells, dist, st))
    for a, b in zip(*out):
        assert torch.equal(a, b)
    return out[0][2].cpu().numpy()


# a cell of `faces` neighbours on a sphere: a slab holds 256 records, a try loads
# 512; rays in a pencil leave half of the faces out, rays all around none
@pytest.mark.parametrize("faces", [255, 256, 257, 300, 511, 512, 513, 600])
@pytest.mark.parametrize("spread", [0.01, 100.0])
def test_long_rows(dev, faces, spread):
    print(f"[gpu-case] one lane, {faces} faces, spread {spread}", flush=True)
    rng = np.random.default_rng(faces)
    sites = np.concatenate([np.zeros((1, 3)), 0.8 * unit(rng.normal(size=(faces, 3)))])
    off = np.concatenate([[0], faces + np.arange(faces + 1)])
    idx = np.concatenate([np.arange(1, faces + 1), np.zeros(faces, int)])
    tex = synth.scene_uniform(faces + 1, 4, seed=3, with_csr=False).texels
    ds = upload(dev, sites, np.full(faces + 1, 0.5), tex, off, idx)
    d = unit(np.array([0.3, -0.5, 0.8]) + spread * rng.normal(size=(200, 3)))
    k = walks(dev, ds, np.zeros((200, 3)), d, np.zeros(200))
    assert (k == 2).all()


# a wave that stands in `cells` cells: 32 rows can be staged
@pytest.mark.parametrize("cells", [1, 2, 31, 32, 33, 64])
@pytest.mark.parametrize("rays", [1, 2, 16, 63, 64, 65, 300])
def test_cells_of_a_wave(dev, cells, rays):
    print(f"[gpu-case] one lane, {rays} rays in {cells} cells", flush=True)
    sc = synth.scene_uniform(200, 4, seed=81)
    ds = upload(dev, sc.sites, sc.density, sc.texels, sc.nbr_off, sc.nbr_idx)
    rng = np.random.default_rng(cells)
    start = rng.permutation(sc.n)[:cells][np.arange(rays) % cells]
    k = walks(dev, ds, sc.sites[start], unit(rng.normal(size=(rays, 3))), start)
    assert rays < 16 or k.max() > 3


@pytest.mark.parametrize("what", ["one site", "two sites", "empty rows", "malformed rows"])
def test_rows_without_faces(dev, what):
    print(f"[gpu-case] one lane, {what}", flush=True)
    sc = synth.scene_uniform(200, 4, seed=91)
    off, idx = sc.nbr_off.astype(np.int64), sc.nbr_idx.astype(np.int64).copy()
    sites, dens, tex = sc.sites, sc.density, sc.texels
    if what == "one site":
        sites, dens, tex, off, idx = sites[:1], dens[:1], tex[:1], [0, 0], np.zeros(0)
    elif what == "two sites":
        sites, dens, tex, off, idx = sites[:2], dens[:2], tex[:2], [0, 1, 2], [1, 0]
    elif what == "empty rows":
        rows = [idx[off[i]:off[i + 1]] if i % 3 else idx[:0] for i in range(sc.n)]
        off, idx = np.concatenate([[0], np.cumsum([len(r) for r in rows])]), np.concatenate(rows)
    else:
        off = off.copy()
        idx[off[3]], idx[off[4]], idx[off[5]] = -1, sc.n + 7, 5
        off[10] = off[11] + 2
    ds = upload(dev, sites, dens, tex, off, idx)
    rng = np.random.default_rng(92)
    n = len(sites)
    # bundles of 32 rays from a cell, then single rays
    start = np.concatenate([np.repeat(rng.integers(0, n, 8), 32), rng.integers(0, n, 77)])
    walks(dev, ds, np.asarray(sites)[start], unit(rng.normal(size=(len(start), 3))), start)


@pytest.mark.parametrize("look", ["map", "full", "sh"])
@pytest.mark.parametrize("tex", ["float32", "float16", "bfloat16"])
@pytest.mark.parametrize("kw", [{}, {"skip_w": 0.02}, {"edge_fp16": 1}])
def test_models_texels_and_schedules(dev, look, tex, kw):
    print(f"[gpu-case] one lane, {look} {tex} {kw}", flush=True)
    sc = synth.scene_uniform(512, 4, seed=95)
    t = {"map": lambda: sc.texels, "full": lambda: synth.full_texels(sc.n, 4, seed=96),
         "sh": lambda: synth.sh_coeffs(sc.n, seed=97)}[look]()
    t = to_dev(np.asarray(t, np.float32), dev)
    if tex != "float32":
        t = voro.voro_cast_texels(t, tex)
    ds = voro.DeviceScene(to_dev(sc.sites, dev), to_dev(sc.density, dev), to_dev(sc.nbr_off, dev),
                          to_dev(sc.nbr_idx, dev), t)
    voro.voro_prepare(ds)
    app = {"map": 0, "full": 1, "sh": 2}[look]
    cam = voro.camera_of(synth.Camera(synth.PINHOLE, 61, 40, synth.look_at(
        (0.1, -0.2, -0.9), (0.2, 0.1, 0.4)), 1.0, 4.0))
    two = dict(kw, lanes_per_ray=2, appearance=app)
    two.pop("edge_fp16", None)    # one lane only; its walk is the exact one
    want = voro.voro_render_views_fwd(ds, [cam], voro.default_params(**two))
    for schedule in (voro.SCHEDULE_GRID, voro.SCHEDULE_PERSISTENT, voro.SCHEDULE_REFILL):
        p = voro.default_params(lanes_per_ray=1, appearance=app, schedule=schedule, **kw)
        got = voro.voro_render_views_fwd(ds, [cam], p)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    o, d, tm = voro.voro_gen_rays([cam], dev)
    s = voro.voro_locate_origins(ds, o[:1]).expand(len(o)).contiguous()
    p = voro.default_params(lanes_per_ray=1, appearance=app, **kw)
    got = voro.voro_render_fwd(ds, o, d, tm, s, p)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
