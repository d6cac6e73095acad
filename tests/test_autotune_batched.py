"""The batched tuner's choice on given timings: the automatic shape is always
among the candidates and stays unless another is clearly faster."""
import types

import pytest
import torch

from paper_2312_00229_amd import autotune

# the strip heights the automatic choice of a batch takes, in either column count
AUTO_ROWS = (8, 16, 24, 32, 48, 64, 96)


def _tune(monkeypatch, auto, time_of):
    """tune_batched with `auto` as the automatic shape and timings time_of(rows, cols)."""
    config = [(0, 0)]

    class Plan:
        def __init__(self, xs, outs, params=None):
            rows, cols = config[0] if config[0] != (0, 0) else auto
            self.plan = types.SimpleNamespace(rows_per_strip=rows, cols_per_lane=cols)

        def run(self):
            pass

    monkeypatch.setattr(autotune, "BatchedZoom", Plan)
    monkeypatch.setattr(autotune, "get_launch_config", lambda: config[0])
    monkeypatch.setattr(autotune, "set_launch_config", lambda r, c: config.__setitem__(0, (r, c)))
    monkeypatch.setattr(autotune, "_warm", lambda fn: None)
    monkeypatch.setattr(autotune, "_time", lambda fn, reps: time_of(*config[0]))
    monkeypatch.setattr(autotune, "_batched_key", lambda xs, outs: "key")
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    rows, cols, times = autotune.tune_batched([torch.zeros(1)], [torch.zeros(1)], use_cache=False)
    assert config[0] == (rows, cols)
    return (rows, cols), times


@pytest.mark.parametrize("cols", [1, 2])
@pytest.mark.parametrize("rows", AUTO_ROWS)
def test_the_automatic_shape_is_a_candidate(monkeypatch, rows, cols):
    best, times = _tune(monkeypatch, (rows, cols), lambda r, c: 1.0 if (r, c) == (rows, cols) else 1.5)
    assert best == (rows, cols) and "%d,%d" % best in times


def test_noise_does_not_replace_the_automatic_shape(monkeypatch):
    times = {(96, 1): 1.01, (64, 2): 1.0}
    assert _tune(monkeypatch, (96, 1), lambda r, c: times.get((r, c), 1.2))[0] == (96, 1)


def test_a_faster_shape_is_taken(monkeypatch):
    times = {(96, 1): 1.10, (64, 2): 1.0}
    assert _tune(monkeypatch, (96, 1), lambda r, c: times.get((r, c), 1.2))[0] == (64, 2)
