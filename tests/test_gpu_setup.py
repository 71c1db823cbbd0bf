"""Set-up kernels at the edges of their workgroups, and the lanes per ray that
the library chooses: cells of the camera centres, texel casts, reordered rows."""
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


# one workgroup's turn is 1,024 sites, 256 workgroups at most; from 262,145
# sites on they have 1,024 threads
@pytest.mark.parametrize("n", [1, 1023, 1025, 5000, 262_145, 300_001])
def test_cells_of_camera_centres(dev, n):
    print(f"[gpu-case] centres n={n}", flush=True)
    rng = np.random.default_rng(n)
    sites = rng.uniform(-1, 1, (n, 3)).astype(np.float32)
    # no neighbours: every ray ends in its start cell, whose colour is its number
    ids = np.arange(n)
    tex = np.zeros((n, 2, 2, 4), np.float32)
    for c in range(3):
        tex[..., c] = (((ids >> (7 * c)) & 127) / 128.0)[:, None, None]
    ds = voro.DeviceScene(torch.from_numpy(sites).to(dev), torch.full((n,), 1e3, device=dev),
                          torch.zeros(n + 1, dtype=torch.int32, device=dev),
                          torch.zeros(0, dtype=torch.int32, device=dev),
                          torch.from_numpy(tex).to(dev))
    voro.voro_prepare(ds)
    eyes = rng.uniform(-1, 1, (16, 3)).astype(np.float32)
    want = [int(((sites.astype(np.float64) - e.astype(np.float64)) ** 2).sum(1).argmin())
            for e in eyes]
    got = voro.voro_locate_origins(ds, torch.from_numpy(eyes).to(dev)).cpu().numpy()
    np.testing.assert_array_equal(got, want)
    cams = [synth.Camera(synth.PINHOLE, 1, 1, synth.look_at(e, e + np.array([0.3, 0.2, 1.0])), 0.5,
                         1.0) for e in eyes.astype(np.float64)]
    for first, views in ((0, cams[:1]), (0, cams), (3, cams[3:8])):   # one scratch for all calls
        rgb, T, _ = voro.voro_render_views_fwd(ds, views)
        d = np.rint(rgb.cpu().numpy() * 128).astype(int)
        np.testing.assert_array_equal(d[:, 0] + (d[:, 1] << 7) + (d[:, 2] << 14),
                                      want[first:first + len(views)])
        assert float(T.max()) == 0.0


# around the ray counts at which the library splits a ray over more lanes
@pytest.mark.parametrize("w,h", [(8, 8), (180, 91), (181, 91), (512, 256), (513, 256)])
def test_default_lanes_give_the_one_lane_walk(dev, w, h):
    print(f"[gpu-case] default lanes {w}x{h}", flush=True)
    ds = voro.device_scene(synth.scene_uniform(512, 4, seed=51), dev)
    voro.voro_prepare(ds)
    cams = [voro.camera_of(synth.Camera(synth.PINHOLE, w, h,
                                        synth.look_at((0, 0, -3), (0, 0, 0)), 1.0, 6.0))]
    g = torch.randn((w * h, 3), device=dev)
    o, d, tm = voro.voro_gen_rays(cams, dev)
    start = voro.voro_locate_origins(ds, o[:1]).expand(len(o)).contiguous()
    out = []
    for lanes in (0, 1):
        p = voro.default_params(lanes_per_ray=lanes)
        rgb, T, _ = voro.voro_render_views_fwd(ds, cams, p)
        rgb2, T2 = voro.voro_render_fwd(ds, o, d, tm, start, p)
        grads = voro.voro_render_views_bwd(ds, cams, rgb, T, None, g, None, p)
        out.append([x.cpu().numpy() for x in (rgb, T, rgb2, T2, *grads)])
    for a, b in zip(out[0][:4], out[1][:4]):
        np.testing.assert_array_equal(a, b)
    for a, b in zip(out[0][4:], out[1][4:]):
        # the same terms summed in another order
        np.testing.assert_allclose(a, b, rtol=0, atol=1e-5 * np.abs(b).max())


@pytest.mark.parametrize("dtype", ["float16", "bfloat16"])
@pytest.mark.parametrize("count,skip", [(1, 0), (7, 0), (8, 0), (9, 0), (1000, 1), (65_541, 0)])
def test_cast_any_length_and_alignment(dev, dtype, count, skip):
    print(f"[gpu-case] cast {dtype} {count} from {skip}", flush=True)
    gen = torch.Generator(device=dev).manual_seed(count)
    src = torch.randn(count + skip, generator=gen, device=dev) * 100.0
    src[-1] = float("inf")
    got = voro.voro_cast_texels(src[skip:], dtype)
    assert torch.equal(got, src[skip:].to(getattr(torch, dtype)))


# rows of 64 cells go to one workgroup; some rows are empty
@pytest.mark.parametrize("n", [1, 63, 64, 65, 200])
def test_reordered_rows(dev, n):
    print(f"[gpu-case] reorder n={n}", flush=True)
    rng = np.random.default_rng(n)
    deg = rng.integers(0, 40, n) * (rng.random(n) < 0.8)
    off = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    idx = rng.integers(0, n, off[-1]).astype(np.int32)
    sites = rng.uniform(-1, 1, (n, 3)).astype(np.float32)
    ds = voro.DeviceScene(*(torch.from_numpy(a).to(dev) for a in (
        sites, np.ones(n, np.float32), off, idx, rng.random((n, 4, 4, 4)).astype(np.float32))))
    out, perm, inv = voro.voro_morton_reorder(ds)
    perm, inv = perm.cpu().numpy(), inv.cpu().numpy()
    q = np.clip(((sites - sites.min(0)) / np.maximum(sites.max(0) - sites.min(0), 1e-30)
                 * np.float32(1024)).astype(int), 0, 1023)
    code = sum(((q[:, a] >> b) & 1) << (3 * b + 2 - a) for a in range(3) for b in range(10))
    np.testing.assert_array_equal(perm, np.argsort(code, kind="stable"))
    np.testing.assert_array_equal(inv[perm], np.arange(n))
    rows = [inv[idx[off[o]:off[o + 1]]] for o in perm]
    np.testing.assert_array_equal(out.nbr_off.cpu().numpy(),
                                  np.concatenate([[0], np.cumsum([len(r) for r in rows])]))
    np.testing.assert_array_equal(out.nbr_idx.cpu().numpy(),
                                  np.concatenate(rows) if len(idx) else idx)
