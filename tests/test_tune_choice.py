"""The tuner's choice (host logic, times drawn at random): noise alone keeps the
default options, whatever the number of candidates; a real gain is taken."""
import random

import pytest

from paper_1209_3314_amd import tune

torch = pytest.importorskip("torch")


class FakeContext:
    def __init__(self):
        self.options = dict(tune.DEFAULTS, wg_waves=8)  # what the caller had set

    def set_options(self, **kw):
        self.options.update(kw)


def choose(monkeypatch, seed, cost):
    rng, ctx = random.Random(seed), FakeContext()
    out = torch.zeros(4)
    noisy = lambda reps: min(cost(ctx.options) * (1.0 + abs(rng.gauss(0.0, 0.02))) for _ in range(reps))
    monkeypatch.setattr(tune, "_timed", lambda fn, reps: noisy(reps))
    got = tune._choose(ctx, lambda: None, [out], tune.GRID["recon"], 3, "the result")
    assert ctx.options == dict(tune.DEFAULTS, wg_waves=8)
    return got


def test_noise_keeps_the_default(monkeypatch):
    kept = 0
    for seed in range(40):
        opts, ms, default_ms = choose(monkeypatch, seed, lambda o: 1.0)
        kept += opts == tune.DEFAULTS
        assert ms <= default_ms
    assert kept >= 39  # by chance one side wins all of 6 turns once in 924


def test_a_gain_is_taken(monkeypatch):
    for seed in range(10):
        opts, ms, default_ms = choose(monkeypatch, seed, lambda o: 0.8 if o["mr_seed_strip"] == 16 else 1.0)
        assert opts["mr_seed_strip"] == 16 and ms < 0.9 * default_ms


def test_a_changed_result_is_an_error(monkeypatch):
    ctx, out = FakeContext(), torch.zeros(4)
    monkeypatch.setattr(tune, "_timed", lambda fn, reps: fn() or 1.0)
    with pytest.raises(RuntimeError):
        tune._choose(ctx, lambda: out.fill_(ctx.options["stage_depth"]) and None, [out], tune.GRID["edt"], 1, "the result")
