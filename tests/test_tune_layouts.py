"""CPU tests of the autotuner's layout stage with a solver that only records
its calls: layouts are timed on whole books, and differences within the noise
leave the first layout."""
import torch

from paper_2606_23367_amd import tune
from paper_2606_23367_amd.solver import to_device
from workloads import make_config

GRID = dict(rho=(3.0,), alpha=(1.8,), check_every=(50,))
LAYOUTS = dict(tile_rows=(0, 1, 2), precision=(1, 0))


class _Recorder:
    def __init__(self):
        self.calls = []

    def solve(self, Q, **cfg):
        self.calls.append((Q.m, cfg))
        return dict(status=torch.zeros(Q.m, dtype=torch.int32))


def _tune(monkeypatch, seconds, sample=4):
    s = _Recorder()
    timed = []

    def fake(solver, Q, cfg):
        timed.append((Q.m, cfg))
        return Q.m, seconds(Q, cfg)

    monkeypatch.setattr(tune, "_timed", fake)
    book = lambda seed: to_device(*make_config("c2", seed, N=40, M=12, k=3, ub=0.2), "cpu")  # noqa: E731
    cfg = tune.autotune(book(0), solver=s, sample=sample, grid=GRID, layouts=LAYOUTS,
                        second=[book(1)], use_cache=False)
    return cfg, s.calls, timed


def test_layouts_are_timed_on_whole_books(monkeypatch):
    cfg, calls, timed = _tune(monkeypatch, lambda Q, cfg: 1.0)
    sized = [m for m, c in calls + timed if "tile_rows" in c]
    assert sized and all(m == 12 for m in sized)
    assert all(m == 4 for m, c in calls + timed if "tile_rows" not in c)


def test_noise_keeps_the_first_layout(monkeypatch):
    # every later layout half a percent faster than the one before
    order = [(t, p) for t in LAYOUTS["tile_rows"] for p in LAYOUTS["precision"]]
    cfg, _, _ = _tune(monkeypatch, lambda Q, cfg: 1.0 - 0.0015 * order.index(
        (cfg["tile_rows"], cfg["precision"])) if "tile_rows" in cfg else 1.0)
    assert (cfg["tile_rows"], cfg["precision"]) == (0, 1)


def test_a_faster_layout_is_taken(monkeypatch):
    cfg, _, _ = _tune(monkeypatch, lambda Q, cfg: 0.9 if cfg.get("tile_rows") == 2 and
                      cfg["precision"] == 0 else 1.0)
    assert (cfg["tile_rows"], cfg["precision"]) == (2, 0)
