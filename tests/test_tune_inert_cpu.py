"""The tuner times a launch shape once, whatever the fields without effect say."""
import types

from paper_0912_3824_amd import tune


class Pool:
    def __init__(self, rebuild_every):
        self.sizes, self.boxes = {0: 1000}, {0: 10.0}
        self.cfg = types.SimpleNamespace(precision=1, rebuild_every=rebuild_every)
        self.shapes = []

    def set_launch(self, **kw):
        self.shapes.append(kw)

    def save(self, slot):
        return b""

    def restore(self, *a):
        pass

    def detach(self, slot):
        pass

    def step(self, n):
        pass


def test_shapes_differing_in_inert_fields_are_timed_once(monkeypatch):
    timed = []
    monkeypatch.setattr(tune, "_time_steps", lambda pool, steps: timed.append(dict(pool.shapes[-1])) or 1.0)
    out = tune.tune(Pool(16), cache=None)
    live = [tuple(v for k, v in s.items() if k not in tune.INERT) for s in timed]
    assert len(live) == len(set(live))
    combinations = 1
    for values in tune.space_for(Pool(16)).values():
        combinations *= len(values)
    assert len(out["all"]) == combinations > len(live)  # each shape is reported
    plain = []
    monkeypatch.setattr(tune, "_time_steps", lambda pool, steps: plain.append(1) or 1.0)
    tune.tune(Pool(0), cache=None)
    assert len(plain) == len(live)
