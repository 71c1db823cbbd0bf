"""Host side of the Python entry points: what a caller keeps in hand is its own."""
import ctypes

import numpy as np
import torch

from paper_2608_17682_amd import synth, voro


def cameras(n):
    return [synth.Camera(synth.PINHOLE, 8 + i, 4, synth.look_at((0, 0, -3), (0, 0, 0)), 1.0, 6.0)
            for i in range(n)]


def test_camera_array_is_a_copy():
    first = voro.camera_array(cameras(3))
    second = voro.camera_array(first)
    second[1].width = 99
    assert [c.width for c in first] == [8, 9, 10]
    assert isinstance(second, ctypes.Array) and [c.width for c in second] == [8, 99, 10]
    assert voro.voro_camera_counts(first) == voro.voro_camera_counts(list(first)) == (108, 108)


def test_scene_counters_are_made_with_the_scene():
    # made when first asked for, they were zeroed on whatever stream that access
    # ran on, and belonged to whatever mode it ran in
    sc = synth.scene_uniform(16, 2, seed=1)
    ds = voro.DeviceScene(*(torch.from_numpy(np.ascontiguousarray(a)) for a in (
        sc.sites, sc.density, sc.nbr_off, sc.nbr_idx, sc.texels)))
    with torch.inference_mode():
        assert ds.stats.tolist() == [0] * voro.STAT_COUNT
    ds.stats += 1
    other = ds.with_arrays(density=ds.density * 2.0)
    assert other.stats is ds.stats and other.stats.tolist() == [1] * voro.STAT_COUNT
