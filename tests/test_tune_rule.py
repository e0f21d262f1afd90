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


@pytest.mark.parametrize("drift", [0.97, 0.995, 1.005, 1.03])
def test_drift_of_the_clock_picks_no_aim(clock, drift):
    """All aims equal, the step time falling or rising from timing to timing: every bucket
    stays in the common launch."""
    clock(lambda b, k: 1.3 * drift ** k)
    assert tune.tune_buckets(SPECS)["best"] == {q: tune._max_waves(q) for q in PRESENT}


def test_one_stray_timing_picks_no_aim(clock):
    clock(lambda b, k: 0.9 if k % 7 == 3 else 1.0)
    assert tune.tune_buckets(SPECS)["best"] == {q: tune._max_waves(q) for q in PRESENT}


def test_a_faster_aim_is_picked(clock):
    """Bucket 5 is 6 % faster at an aim of 2, under a drift."""
    clock(lambda b, k: 1.3 * 1.01 ** k * (0.94 if b.waves.get(5) == 2 else 1.0))
    r = tune.tune_buckets(SPECS)
    assert r["best"] == {q: 2 if q == 5 else tune._max_waves(q) for q in PRESENT}
    assert sorted(r["ms"][5]) == [1, 2, 3]


def test_unit_pairs_are_not_chosen_by_timing(clock):
    """The library ignores the pairs: the timings' noise must not pick among them."""
    clock(lambda b, k: 1.3 * 0.97 ** k)
    r = tune.tune_group(SPECS)
    assert r["best"] == tune.GROUP_DEFAULT and not r["cached"]
    assert set(r["ms"]) == set(tune.GROUP_CANDIDATES) and len(set(r["ms"].values())) == 1
    clock(lambda b, k: 1.3 * 1.03 ** k)
    assert tune.tune_group(SPECS, candidates=(4, 2), use_cache=False)["best"] == 4
    assert tune.tune_group(SPECS)["cached"]
