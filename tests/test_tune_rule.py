"""The autotuner's choices, with the device's timings replaced by made-up ones."""
import json

import pytest

from paper_1905_10252_amd import tune

SPECS = [dict(n=1000, d=d, mean=None, chol=None, seed=1, sampler_id=k, rw_sd=0.1)
         for k, d in enumerate((3, 20, 44, 60))]
PRESENT = [0, 2, 5, 7]


class FakeBatch:
    def __init__(self):
        self.waves = {}

    def set_group(self, pairs):
        pass

    def set_bucket_waves(self, q, w):
        self.waves[q] = w


@pytest.fixture
def clock(monkeypatch, tmp_path):
    """Sets the step time as a function of (batch, number of timings so far)."""
    monkeypatch.setenv("SMC_TUNE_CACHE", str(tmp_path / "tune.json"))
    monkeypatch.setattr(tune, "arch", lambda dev: "gfx950")
    monkeypatch.setattr(tune, "_scratch_batch", lambda specs, dev: FakeBatch())
    calls = []

    def use(fn):
        def time_steps(b, steps):
            calls.append(dict(b.waves))
            return fn(b, len(calls) - 1)
        monkeypatch.setattr(tune, "_time_steps", time_steps)
    use.calls = calls
    use.path = tmp_path / "tune.json"
    return use


def test_entries_of_an_earlier_rule_are_not_reused(clock):
    """An aim chosen when every bucket had a launch of its own would take the bucket out
    of the common one."""
    old = {"k_bquad|waves|%d|gfx950|%s" % (q, tune.workload_digest(SPECS)):
           {"best": 1, "ms": {"1": 1.0}} for q in range(8)}
    clock.path.write_text(json.dumps(old))
    clock(lambda b, k: 1.0)
    r = tune.tune_buckets(SPECS)
    assert r["cached"] == []
    assert r["best"] == {q: tune._max_waves(q) for q in PRESENT}
    r2 = tune.tune_buckets(SPECS)
    assert r2["cached"] == PRESENT and r2["best"] == r["best"]
