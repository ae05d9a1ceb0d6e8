"""The autotuner's sweep cap is for the sweeps (with an adaptive dimension, in the
memory-saving variant, under capture, on grids too large for resident launches):
it times those, on grids that take resident launches too."""


def test_tune_single_times_sweeps(monkeypatch, tmp_path):
    import torch
    from paper_1407_7370_amd import autotune, binding

    class Stub:
        cost = {1: 3.0, 2: 1.0, 3: 2.0}

        def __init__(self, *a):
            self.cap = self.wait = None

        def set_wait(self, seconds):
            self.wait = seconds

        def set_launch(self, c):
            self.cap = c
            return c

        def step(self, *a, **kw):
            assert self.wait == 0.0, "a resident launch would be timed"

        def close(self):
            pass

    made = []
    monkeypatch.setattr(binding, "Propagator", lambda *a: made.append(Stub()) or made[-1])
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setattr(autotune, "device_arch", lambda: "gfx950")
    monkeypatch.setattr(autotune, "_time_steps", lambda step, n: (step(n), Stub.cost[made[-1].cap])[1])
    cache = str(tmp_path / "tune.json")
    prob = dict(nx=64, ny=48, bc_y=0, bz=0.0, pot_kind=0)
    out = autotune.tune_single(prob, torch.zeros(2), 12, "fp64", 1e-3, candidates=(1, 2, 3), cache=cache)
    assert out["best"] == 2 and len(made) == 1
    assert autotune.lookup(autotune.key_single(prob, 12, "fp64", "gfx950"), cache) == 2
