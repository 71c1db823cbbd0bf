"""Forward kernels with one lane per ray, which stage the edge rows of a wave's
cells: around the ray count from which they are held to a fifth wave per SIMD,
against two lanes per ray, which stage nothing, bit by bit."""
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
