"""Brute-force search for the cells of origins and camera centres, at the sizes
where its split changes: chunks of 1,024 and 4,096 sites, one chunk to many, one
kernel with tickets or two, workgroups of 256 and 1,024 threads, wide and narrow
turns.  Every site lies twice in the scene: ties go to the smaller index."""
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


def scene(n, dev):
    """n cells without neighbours, whose colour is their number (see cell_of)."""
    rng = np.random.default_rng(n)
    half = rng.uniform(-1, 1, ((n + 1) // 2, 3)).astype(np.float32)
    sites = np.concatenate([half, half])[:n]
    ids = np.arange(n)
    tex = np.zeros((n, 2, 2, 4), np.float32)
    for c in range(3):
        tex[..., c] = (((ids >> (8 * c)) & 255) / 256.0)[:, None, None]
    ds = voro.DeviceScene(torch.from_numpy(sites).to(dev), torch.full((n,), 1e3, device=dev),
                          torch.zeros(n + 1, dtype=torch.int32, device=dev),
                          torch.zeros(0, dtype=torch.int32, device=dev),
                          torch.from_numpy(tex).to(dev))
    voro.voro_prepare(ds)
    return sites, ds, rng


def nearest(sites, o):
    d = sites.astype(np.float64) - o.astype(np.float64)
    return int((d[:, 0] ** 2 + d[:, 1] ** 2 + d[:, 2] ** 2).argmin())


@pytest.mark.parametrize("n,U", [
    (1, 64), (2, 1), (1024, 64), (1025, 64),          # one chunk, two
    (8192, 64), (8193, 64),                           # 8 chunks; 9, rounded up to 16
    (16_384, 64), (16_385, 64),                       # 16 of 1,024; of 4,096
    (262_144, 4), (262_145, 5),                       # 256 chunks of 1,024; 72 of 4,096
    (1_048_576, 1), (1_048_577, 1),                   # 256 and 1,024 threads
    (3_145_728, 8), (3_145_729, 8), (3_145_729, 7),   # wide, narrow, wide turns
])
def test_cells_of_origins(dev, n, U):
    print(f"[gpu-case] locate n={n} U={U}", flush=True)
    sites, ds, rng = scene(n, dev)
    o = rng.uniform(-1, 1, (U, 3)).astype(np.float32)
    got = voro.voro_locate_origins(ds, torch.from_numpy(o).to(dev)).cpu().numpy()
    np.testing.assert_array_equal(got, [nearest(sites, x) for x in o])


@pytest.mark.parametrize("n,V", [(16_384, 16), (16_385, 16), (32_768, 8), (32_769, 8),
                                 (262_145, 1), (262_145, 2), (1_048_577, 1), (3_145_729, 8)])
@pytest.mark.parametrize("schedule", [voro.SCHEDULE_GRID, voro.SCHEDULE_PERSISTENT])
def test_cells_of_camera_centres_on_either_route(dev, n, V, schedule):
    print(f"[gpu-case] centres n={n} V={V} schedule={schedule}", flush=True)
    sites, ds, rng = scene(n, dev)
    p = voro.default_params(schedule=schedule)
    # three launches on one scratch: each has to find its queue and ticket at zero
    for views in (V, max(1, V // 2), V):
        eyes = rng.uniform(-1, 1, (views, 3)).astype(np.float32)
        cams = [synth.Camera(synth.PINHOLE, 9, 7, synth.look_at(e, e + np.array([0.3, 0.2, 1.0])),
                             0.5, 1.0) for e in eyes.astype(np.float64)]
        rgb, T, _ = voro.voro_render_views_fwd(ds, cams, p)
        d = np.rint(rgb.cpu().numpy() * 256).astype(int).reshape(views, 63, 3)
        got = d[..., 0] + (d[..., 1] << 8) + (d[..., 2] << 16)
        np.testing.assert_array_equal(got, np.array([nearest(sites, e) for e in eyes])[:, None]
                                      + np.zeros((1, 63), int))
        assert float(T.max()) == 0.0
