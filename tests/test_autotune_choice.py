"""The autotuner's choice, with the timings given (no GPU): lds_tiles changes nothing, so a
timing that happens to be lower with it is noise and not a winner."""
from types import SimpleNamespace

from paper_1804_03479_amd import autotune


class Level:
    def __init__(self):
        self.cfg = SimpleNamespace(scheme=1, recon=1, riemann=2, prec=1)
        self.launch = (0, 0, 0, 0)

    def set_launch(self, *shape):
        self.launch = shape


def test_the_tile_option_is_never_the_winner(tmp_path, monkeypatch):
    level = Level()
    h = SimpleNamespace(solvers=[level], levels=[SimpleNamespace(groups=None)],
                        set_launch=lambda shapes: level.set_launch(*shapes[0]))
    times = {0: 3.0, 1: 2.0, 4: 2.5}
    monkeypatch.setattr(autotune, "level_key", lambda h, lvl: "level")
    monkeypatch.setattr(autotune, "time_level", lambda h, lvl, reps: times[level.launch[0]] - 0.01 * level.launch[3])
    r = autotune.tune(h, candidates=(0, 1, 4), cache=str(tmp_path / "tune.json"))
    assert r["candidates"] == [[(0, 0, 0, 0), (1, 0, 0, 0), (4, 0, 0, 0), (1, 0, 0, 1)]]
    assert r["ms"] == [[3.0, 2.0, 2.5, 1.99]]
    assert r["shapes"] == [(1, 0, 0, 0)] and level.launch == (1, 0, 0, 0)
    again = autotune.tune(h, candidates=(0, 1, 4), cache=str(tmp_path / "tune.json"), use_cache=True)
    assert again["shapes"] == r["shapes"]
