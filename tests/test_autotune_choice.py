"""What the autotuner makes of given timings (CPU: a sweep whose times are a
table): a choice is never slower, by whole untimed runs, than any one shape on
every level."""
import json
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")

# ms of whole runs with one shape on both levels (one launch over item queues
# where the shape has a persistent kernel), of the levels' own launches in a
# timed run, and of a run with a shape for each level (a launch per job)
WHOLE = {(4, 4): 12.8, (8, 4): 14.0, (2, 8): 15.4}
LEVELS = {(4, 4): (5.0, 10.2), (8, 4): (7.0, 11.0), (2, 8): (6.0, 9.0)}


class Sweep:
    """A grid config of two levels; (4, 8) is not compiled."""

    def __init__(self, mixed, launch=0, levels=2):
        self.settings = SimpleNamespace(levels=[None] * levels)
        self.cfg = SimpleNamespace(launch=launch)
        self.mixed, self.timing, self.tiles, self.chunks, self.ctx = mixed, False, [(4, 4)] * levels, [0] * levels, self

    def set_tile(self, l, r, w):
        self.tiles[l] = (r, w)

    def set_chunks(self, l, c):
        self.chunks[l] = c

    def set_timing(self, on):
        self.timing = on

    def run(self, frames, outputs):
        if (4, 8) in self.tiles:
            raise RuntimeError("no kernel")
        if self.timing:   # read after the run, whether or not timing is still on
            self.last = [LEVELS[t][l] for l, t in enumerate(self.tiles)]

    def whole(self):
        self.run(None, None)
        assert not self.timing, "whole runs are not timed launch by launch"
        one = all(t == self.tiles[0] for t in self.tiles)
        return (WHOLE[self.tiles[0]] if one else self.mixed) + 0.1 * sum(c not in (0, 4) for c in self.chunks)

    def times(self):
        return self.last

    def sweep_kernel_ms(self):   # the mean over the launches, and their number
        return sum(self.last) / len(self.last), len(self.last)


@pytest.fixture
def tuner(monkeypatch):
    from paper_1809_06132_amd import autotune, psweep

    class Event:   # of the two events of one timed run, the second knows its time
        def __init__(self, **_):
            pass

        def record(self):
            pass

        def elapsed_time(self, other):
            return current[0].whole()

    current = [None]
    monkeypatch.setattr(torch.cuda, "Event", Event)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setattr(autotune, "_key", lambda sweep, frames: "key")
    monkeypatch.setattr(psweep, "psweep_sweep_kernel_times", lambda ctx: ctx.times())

    def tune(sweep, **kw):
        current[0] = sweep
        return autotune.tune(sweep, [None], [None], reps=2, candidates=[(4, 4), (4, 8), (8, 4), (2, 8)], **kw)
    return tune


@pytest.mark.parametrize("mixed,tiles", [(14.9, [[4, 4], [4, 4]]), (12.0, [[4, 4], [2, 8]])])
def test_mix_of_shapes_only_where_its_run_is_faster(tuner, tmp_path, mixed, tiles):
    s = Sweep(mixed)
    cache = tmp_path / "tiles.json"
    choice = tuner(s, cache_path=str(cache))
    assert choice["tiles"] == tiles and s.tiles == [tuple(t) for t in tiles]
    assert s.whole() <= min(WHOLE.values()) and not s.timing
    assert choice["candidates"]["4x8"] == float("inf") and choice["candidates"]["mix"] == mixed
    assert json.loads(cache.read_text())["key"]["tiles"] == tiles
    again = Sweep(mixed)
    assert tuner(again, cache_path=str(cache))["tiles"] == tiles and again.tiles == s.tiles


def test_one_level_is_ranked_by_whole_runs(tuner):
    s = Sweep(99.0, levels=1)
    assert tuner(s, cache_path=None)["tiles"] == [[4, 4]] and s.chunks == [0]


def test_persistent_config_is_ranked_by_its_launch(tuner):
    s = Sweep(99.0, launch=1)
    # sums of the levels' times: 15.2, 18.0 and 15.0
    assert tuner(s, cache_path=None)["tiles"] == [[2, 8], [2, 8]]


def test_key_sets_choices_ranked_otherwise_apart(monkeypatch):
    """Choices cached before whole runs ranked the shapes are not taken."""
    from paper_1809_06132_amd import autotune
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda d: SimpleNamespace(gcnArchName="gfx950"))
    lv = SimpleNamespace(n_fronto=3, n_ground=0, window=7, downsample=1, crop=(0, 0, 0, 0))
    sweep = SimpleNamespace(device="cuda:0", settings=SimpleNamespace(levels=[lv]), cfg=SimpleNamespace(storage=0, launch=0))
    key = autotune._key(sweep, [{"ref": torch.zeros(4, 6), "srcs": [None]}])
    assert key == "gfx950|3+0w7d1c(0, 0, 0, 0)|S1|st0|launch0|6x4|runs"
