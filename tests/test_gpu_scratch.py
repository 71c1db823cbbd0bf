"""Scratch of a multi-view launch: the ticket that counts the workgroups of the
camera-centre search is zero again after every launch, whatever the launch
found there, so that one spoiled call (two calls that overlap on one workspace)
does not spoil those that follow."""
import numpy as np
import pytest
import torch

from paper_2608_17682_amd import synth, voro

pytestmark = pytest.mark.gpu

N = 5000            # five workgroups search them (1,024 sites each)
SCHEDULES = {"grid": voro.SCHEDULE_GRID, "persistent": voro.SCHEDULE_PERSISTENT,
             "refill": voro.SCHEDULE_REFILL}


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    voro.lib()
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def scene():
    return synth.scene_uniform(N, 4, seed=61)


def prepared(scene, dev):
    ds = voro.device_scene(scene, dev)
    voro.voro_prepare(ds)
    return ds


def ticket(ds):
    """The ticket's word: 64 bytes into the counters, the 4,096 bytes in front of
    the per-cell accumulator (16 bytes a cell, at the workspace's end)."""
    at = voro.voro_workspace_size(ds) - (16 * ds.n + 255) // 256 * 256 - 4096 + 64
    return ds.ws[at:at + 4].view(torch.int32)


def camera(eye):
    return voro.camera_of(synth.Camera(synth.PINHOLE, 40, 24, synth.look_at(eye, (0, 0, 0)), 1.0,
                                       3.0))


# 3 early tickets, all of them, and more than there are workgroups
@pytest.mark.parametrize("left", [3, 5, 1000])
@pytest.mark.parametrize("spoiled", ["grid", "persistent", "refill", "bwd"])
def test_ticket_left_over_spoils_one_call_at_most(dev, scene, left, spoiled):
    print(f"[gpu-case] ticket left={left} spoiled={spoiled}", flush=True)
    first, second = camera((0.8, 0.1, -0.6)), camera((-0.5, 0.7, 0.3))
    want = voro.voro_render_views_fwd(prepared(scene, dev), [second])[0]
    ds = prepared(scene, dev)
    # a good call first: the partial results and centre cells are a scene's own
    rgb, T, _ = voro.voro_render_views_fwd(ds, [first])
    assert int(ticket(ds)) == 0
    ticket(ds).fill_(left)
    if spoiled == "bwd":
        voro.voro_render_views_bwd(ds, [first], rgb, T, None, torch.ones_like(rgb))
    else:
        voro.voro_render_views_fwd(ds, [first], voro.default_params(schedule=SCHEDULES[spoiled]))
    assert int(ticket(ds)) == 0
    for schedule in SCHEDULES.values():
        got = voro.voro_render_views_fwd(ds, [second], voro.default_params(schedule=schedule))[0]
        np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
        assert int(ticket(ds)) == 0
