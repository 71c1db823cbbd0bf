"""The staged rows of the forward walk leave out the faces that point away from
every ray of the wave: narrow, wide and ragged tiles against the walk that
searches whole rows (two lanes per ray), bit by bit."""
import numpy as np
import pytest
import torch

from paper_2608_17682_amd import synth, voro

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ds():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # a coarse scene: the rays of a tile share cells, so rows are staged
    d = voro.device_scene(synth.scene_uniform(512, 4, seed=41), torch.device("cuda:0"))
    voro.voro_prepare(d)
    return d


# fields of view from a pencil of rays to more than a half space in one tile
@pytest.mark.parametrize("model,fov", [(synth.PINHOLE, 0.01), (synth.PINHOLE, 1.0),
                                       (synth.PINHOLE, 3.1), (synth.FISHEYE, 6.2),
                                       (synth.THIN_LENS, 1.0)])
@pytest.mark.parametrize("size", [(8, 8), (9, 7), (61, 40)])
@pytest.mark.parametrize("schedule", [voro.SCHEDULE_GRID, voro.SCHEDULE_PERSISTENT])
def test_culled_rows_give_the_same_walk(ds, model, fov, size, schedule):
    print(f"[gpu-case] cull model={model} fov={fov} size={size} schedule={schedule}", flush=True)
    cam = synth.Camera(model, *size, synth.look_at((0.1, -0.2, -0.9), (0.2, 0.1, 0.4)), fov, 4.0,
                       lens_radius=0.2, focus_dist=1.0, spp=4 if model == synth.THIN_LENS else 1)
    n = cam.n_rays
    out = []
    for lanes in (1, 2):
        k = torch.zeros(n, dtype=torch.int32, device="cuda")
        p = voro.default_params(lanes_per_ray=lanes, schedule=schedule)
        rgb, T, _ = voro.voro_render_views_fwd(ds, [cam], p, nsteps=k)
        torch.cuda.synchronize()
        out.append([x.cpu().numpy() for x in (rgb, T, k)])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    assert out[0][2].max() > 3
