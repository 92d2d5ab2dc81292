"""The autotuner's choice of launch against a clock that the test sets: the
library's own shape (all zeros) is timed over every grid and returned where it is
fastest, and a cached choice is used only over the grid it was made with."""
import json

import pytest

from paper_2305_01867_amd import autotune


@pytest.fixture
def clock(monkeypatch):
    """Events that read a clock which run() advances."""
    now = [0.0]

    class Event:
        def __init__(self, enable_timing):
            self.at = None

        def record(self, stream):
            self.at = now[0]

        def synchronize(self):
            pass

        def elapsed_time(self, other):
            return other.at - self.at

    monkeypatch.setattr(autotune.torch.cuda, "Event", Event)
    monkeypatch.setattr(autotune.torch.cuda, "current_stream", lambda: None)
    return now


def _own(c):
    return c.get("block", 0) == c.get("stack_depth", 0) == c.get("waves_per_cu", 0) == 0


@pytest.mark.parametrize("space", [None, {"block": (256, 1024), "stack_depth": (12, 20), "ray_sort": (0, 1)},
                                   {"ray_sort": (0, 2), "node_width": (0, 2)}])
def test_the_library_s_own_shape_is_timed_and_returned_where_it_is_fastest(clock, space):
    def run(**c):
        clock[0] += 1.0 if _own(c) and c["ray_sort"] == 0 and not c.get("node_width") else 4.0

    best, timings = autotune.tune(run, "k", None, space=space, reps=2)
    assert _own(best) and best["ray_sort"] == 0 and best["ms"] == 1.0
    choices = [tuple(sorted((k, v) for k, v in t.items() if k != "ms")) for t in timings]
    assert len(set(choices)) == len(choices)
    for sort in (space or autotune.SPACE)["ray_sort"]:
        assert any(_own(t) and t["ray_sort"] == sort for t in timings)


def test_the_fastest_shape_is_returned_where_it_is_not_the_library_s(clock):
    def run(**c):
        clock[0] += 1.0 if (c["block"], c["stack_depth"]) == (256, 12) else 2.0

    best, _ = autotune.tune(run, "k", None, space={"block": (256, 512), "stack_depth": (12, 20)})
    assert (best["block"], best["stack_depth"]) == (256, 12)


def test_a_choice_cached_over_another_grid_is_made_again(clock, tmp_path):
    path = str(tmp_path / "tune.json")
    with open(path, "w") as fh:  # as written before the grid was kept beside the choice
        json.dump({"k": {"block": 256, "stack_depth": 12, "ms": 3.0}}, fh)

    def run(**c):
        clock[0] += 1.0 if _own(c) else 2.0

    best, timings = autotune.tune(run, "k", path)
    assert timings is not None and _own(best)
    again, none = autotune.tune(run, "k", path)
    assert again == best and none is None
    other, timings = autotune.tune(run, "k", path, space={"block": (64,)})
    assert timings is not None and other["block"] == 0
