"""What the autotuner times (CPU, with a stand-in for the rig and the clock):
the default split always, whatever the height of the blocks, and no two
settings that give the same work; and that choices timed on other splits are
not taken from the cache."""
import os

import pytest

from paper_1910_03517_amd import autotune, rt


class FakeRig:
    def __init__(self, cams, n_blocks):
        self.cams, self.opts, self.split, self.seen = cams, rt.Options(n_blocks=n_blocks), autotune.DEFAULT_SPLIT, []

    def tune(self, tile_rows, grid=0):
        self.split = (tile_rows, grid)
        self.seen.append(self.split)


def cams_of(w, h, n=1):
    return [rt.Camera(w, h, 3, 8, 0, p).with_pitch() for p in range(n)]


@pytest.fixture
def clock(monkeypatch):
    us = {}
    monkeypatch.setattr(autotune, "device_arch", lambda: "gfx950")
    monkeypatch.setattr(autotune, "time_frameset", lambda rig, frames, outs, iters=30: us.get(rig.split, 50.0))
    return us


@pytest.mark.parametrize("w,h,nb", [(640, 480, 16), (640, 40, 4), (1920, 1080, 64), (1920, 1080, 16), (320, 8, 16)])
def test_default_split_is_timed_and_kept_when_fastest(clock, tmp_path, w, h, nb):
    clock[autotune.DEFAULT_SPLIT] = 10.0
    rig = FakeRig(cams_of(w, h), nb)
    best = autotune.tune(rig, [None], [None], cache_path=os.path.join(tmp_path, "c.json"))
    assert (best.tile_rows, best.grid) == autotune.DEFAULT_SPLIT == rig.split
    timed = rig.seen[:-1]
    assert len(timed) == len(set(timed))
    assert sorted(g for _, g in timed if g) == sorted(g for g in autotune.GRIDS if g)     # each number of workgroups once
    again = FakeRig(cams_of(w, h), nb)
    assert autotune.apply_cached(again, os.path.join(tmp_path, "c.json")) is not None


def test_default_split_value_is_the_contexts(clock):
    """rt_ctx_create's own split is the one the tuner calls the default."""
    src = open(os.path.join(os.path.dirname(rt.__file__), "csrc", "rt_api.hip")).read()
    assert f"constexpr int kDefaultTileRows = {autotune.DEFAULT_SPLIT[0]};" in src
    assert autotune.DEFAULT_SPLIT[1] == 0
    assert autotune.DEFAULT_SPLIT in autotune.PIPE_SPLITS


def test_choices_of_other_splits_are_not_taken(clock, tmp_path, monkeypatch):
    path = os.path.join(tmp_path, "c.json")
    monkeypatch.setattr(autotune, "SPLIT_VERSION", autotune.SPLIT_VERSION - 1)
    autotune.tune(FakeRig(cams_of(640, 480), 16), [None], [None], cache_path=path)
    monkeypatch.undo()
    monkeypatch.setattr(autotune, "device_arch", lambda: "gfx950")
    assert autotune.apply_cached(FakeRig(cams_of(640, 480), 16), path) is None
    assert autotune.cached_pipe(FakeRig(cams_of(640, 480), 16), path) is None


def test_given_candidates_alone_are_timed(clock, tmp_path):
    rig = FakeRig(cams_of(640, 480), 16)
    autotune.tune(rig, [None], [None], cache_path=None, cands=[(8, 0), (16, 1024)])
    assert rig.seen[:-1] == [(8, 0), (16, 1024)]
