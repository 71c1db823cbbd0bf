"""params_for: which launches take their shape from the tuning table."""
import json
from types import SimpleNamespace

import pytest

from paper_2608_17682_amd import autotune, synth, voro

DS = SimpleNamespace(n=100_000, tex_res=8, tex_dtype=voro.TEX_F32)


@pytest.fixture
def table(tmp_path, monkeypatch):
    def write(**entries):
        keep = {autotune.workload_key(n, 8, voro.TEX_F32, [synth.PINHOLE], d): e
                for (n, d), e in ((k.split("_"), e) for k, e in entries.items())
                for n in [int(n[1:])]}
        monkeypatch.setattr(autotune, "TABLE", str(tmp_path / "table.json"))
        (tmp_path / "table.json").write_text(json.dumps(keep))
    return write


def shape(rays, direction):
    cam = synth.Camera(synth.PINHOLE, rays, 1, synth.look_at((0, 0, -3), (0, 0, 0)), 1.0, 6.0)
    p = autotune.params_for(DS, [cam], direction)
    return p.lanes_per_ray, p.tile_w, p.tile_h


LARGE = {"lanes_per_ray": 1, "tile_w": 16, "tile_h": 4, "rays": 1_000_000}
SMALL = {"lanes_per_ray": 4, "tile_w": 4, "tile_h": 4, "rays": 20_000}
PLAIN = {"lanes_per_ray": 2, "tile_w": 8, "tile_h": 4}     # does not say
DEFAULT = (0, 0, 0)


@pytest.mark.parametrize("direction,most", [("fwd", 1 << 17), ("bwd", 1 << 16)])
def test_small_launches_take_entries_tuned_on_small_launches(table, direction, most):
    table(**{f"n100000_{direction}": SMALL})
    assert shape(most, direction) == (4, 4, 4) == shape(most + 1, direction)
    table(**{f"n100000_{direction}": LARGE})
    assert shape(most, direction) == DEFAULT and shape(most + 1, direction) == (1, 16, 4)
    table(**{f"n100000_{direction}": PLAIN})
    assert shape(most, direction) == (2, 8, 4) == shape(most + 1, direction)
    # the nearest scene among those that count
    table(**{f"n100000_{direction}": LARGE, f"n400000_{direction}": SMALL})
    assert shape(most, direction) == (4, 4, 4) and shape(most + 1, direction) == (1, 16, 4)


def test_cameras_of_any_iterable(table):
    table(n100000_fwd=LARGE)
    cam = synth.Camera(synth.PINHOLE, 1000, 1000, synth.look_at((0, 0, -3), (0, 0, 0)), 1.0, 6.0)
    for cams in ([cam], (c for c in [cam]), iter((cam,))):
        p = autotune.params_for(DS, cams, "fwd")
        assert (p.lanes_per_ray, p.tile_w, p.tile_h) == (1, 16, 4)


def test_committed_entries_come_from_the_tuner():
    tried = {"fwd": autotune.candidates(),
             "bwd": [c for c in autotune.candidates() if c["schedule"] != voro.SCHEDULE_REFILL]}
    for key, e in autotune._load().items():
        shapes = tried[key.split("|")[-1]]
        assert {k: e[k] for k in autotune.LAUNCH_FIELDS} in shapes, key
        assert e["candidates"] == len(shapes), key


def test_table_is_the_files_present_text(table):
    table(n100000_fwd=LARGE)
    assert shape(1 << 18, "fwd") == (1, 16, 4)
    autotune._load().clear()           # a caller's copy
    assert shape(1 << 18, "fwd") == (1, 16, 4)
    table(n100000_fwd=dict(LARGE, tile_w=32, tile_h=2))     # as long a text
    assert shape(1 << 18, "fwd") == (1, 32, 2)
