"""The adjoint's record merge and gradient table on the GPU: more distinct
keys in a wave than one matrix product holds, more keys in a workgroup than
its table, texture sides that are no power of two, and records that are not
finite."""
import numpy as np
import pytest
import torch

from oracle import batch, walk
from paper_2608_17682_amd import synth, voro
from helpers import f32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    voro.lib()
    return torch.device("cuda:0")


def rays_in(scene, n, seed):
    """n rays from random points in random directions: no two of a wave alike."""
    rng = np.random.default_rng(seed)
    o = f32(rng.uniform(-0.9, 0.9, (n, 3)))
    d = rng.normal(size=(n, 3))
    d = f32(d / np.linalg.norm(d, axis=1, keepdims=True))
    tm = np.full(n, 1.5, np.float32)
    starts = np.array([walk.nearest_site(scene.sites, x)[0] for x in o], np.int32)
    ref = batch.evaluate(scene.sites.astype(np.float64), scene.density, scene.texels, o, d, tm,
                         starts=starts, keep_records=np.ones(n, bool), workers=1)
    return o, d, tm, starts, ref


def gradients(dev, scene, o, d, tm, starts, g_rgb, g_T, lpr, cap=0):
    ds = voro.device_scene(scene, dev)
    voro.voro_prepare(ds)
    O, D, TM, S, G, GT = (torch.from_numpy(np.ascontiguousarray(x)).to(dev)
                          for x in (o, d, tm, starts, g_rgb, g_T))
    p = voro.default_params(lanes_per_ray=lpr)
    trace = torch.empty((cap, len(o), 2), dtype=torch.int32, device=dev) if cap else None
    rgb, T = voro.voro_render_fwd(ds, O, D, TM, S, p, trace=trace)
    out = voro.voro_render_bwd(ds, O, D, TM, S, rgb, T, G, GT, p, trace=trace)
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in out]


# 700 rays of 16x16 texels hold some thousands of (cell, quad) keys per
# workgroup (its table has 512 entries); 63 and 65 end a wave early and late
@pytest.mark.parametrize("n,res,lpr,cap", [(1, 4, 1, 0), (63, 3, 1, 4), (65, 5, 2, 0),
                                           (300, 7, 1, 64), (700, 16, 1, 3), (700, 16, 4, 0)])
def test_scattered_records_match_oracle(dev, n, res, lpr, cap):
    scene = synth.scene_uniform(512, res, seed=31)
    print(f"[gpu-case] merge n={n} res={res} lanes={lpr} stored={cap}", flush=True)
    o, d, tm, starts, ref = rays_in(scene, n, 32)
    g_rgb, g_T = synth.upstream(n, 33)
    g_rgb[ref["degenerate"]] = 0.0
    g_T[ref["degenerate"]] = 0.0
    got = gradients(dev, scene, o, d, tm, starts, g_rgb, g_T, lpr, cap)
    ids, *want = batch.sparse_gradients(scene.sites, scene.density, scene.texels, o, d, tm,
                                        ref["records"], g_rgb, g_T)
    # records are products of a few FP32 factors: 1e-4 of the largest component + 1e-6
    for a, w in zip(got, want):
        full = np.zeros(a.shape)
        full[ids] = w
        np.testing.assert_allclose(a, full, rtol=0, atol=1e-4 * np.abs(full).max() + 1e-6)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_nonfinite_record_stays_in_its_cells(dev, bad):
    # one ray's upstream gradient is not finite: every cell that this ray does
    # not reach keeps the gradient of the other rays, in the same waves
    scene = synth.scene_uniform(512, 4, seed=31)
    print(f"[gpu-case] merge upstream {bad}", flush=True)
    n = 300
    o, d, tm, starts, ref = rays_in(scene, n, 34)
    g_rgb, g_T = synth.upstream(n, 35)
    g_rgb[17] = 0.0
    g_T[17] = 0.0
    want = gradients(dev, scene, o, d, tm, starts, g_rgb, g_T, 1)
    g_rgb[17, 1] = bad
    got = gradients(dev, scene, o, d, tm, starts, g_rgb, g_T, 1)
    touched = np.zeros(scene.n, bool)
    for c in ref["cells"][17]:
        touched[c] = True
        touched[scene.nbr_idx[scene.nbr_off[c]:scene.nbr_off[c + 1]]] = True
    assert not np.isfinite(got[1][touched]).all() and not touched.all()
    for a, w in zip(got, want):
        # the same FP32 sums in another order: n terms of eps / 2 each
        np.testing.assert_allclose(a[~touched], w[~touched], rtol=0,
                                   atol=n * 2.0 ** -24 * np.abs(w).max())
