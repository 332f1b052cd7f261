"""Settling one knob of a recorded setting over several batches."""

from __future__ import annotations

import json
import os

import pytest

from paper_1807_02119_amd import tune


def test_settle_takes_the_least_mean_and_times_it():
    best = dict(tune.DEFAULTS, split_min_log2=13, buckets={"2": {"gemm_tasks_log2": 4}})
    rec = {"best": best, "best_ms": 1.0, "confirm": {"best_median_ms": 1.0}, "default_ms": 2.0,
           "plan_wide": {}, "table": [dict(best, ms=1.0)]}
    seen = []

    def measure(seed):
        def m(flat):
            s = tune.split_setting(flat)
            if s == tune.DEFAULTS:
                return 2.5
            assert s["buckets"] == {"2": {"gemm_tasks_log2": 4}}
            seen.append((seed, s["split_min_log2"]))
            # the searched batch is a little slower with 10, the others much faster
            return {13: 1.0, 10: 1.1}[s["split_min_log2"]] if seed == 0 else \
                {13: 0.9, 10: 0.6}[s["split_min_log2"]]
        return m

    out = tune.settle(rec, "split_min_log2", [13, 10], {s: measure(s) for s in (0, 101, 102)},
                      log=lambda m: None)
    assert set(seen) == {(s, v) for s in (0, 101, 102) for v in (13, 10)}
    assert out["best"] == dict(best, split_min_log2=10)
    assert out["best_ms"] == out["confirm"]["best_median_ms"] == 1.1
    assert out["default_ms"] == 2.5
    assert out["settled"]["mean_ms"]["10"] == pytest.approx(2.3 / 3)
    assert out["searched"]["best"] == best and out["searched"]["best_ms"] == 1.0
    assert dict(out["best"], ms=1.1) in out["table"] and dict(best, ms=1.0) in out["table"]


@pytest.mark.parametrize("workload", ["q3_200_600", "batched"])
def test_recorded_settings_were_timed(workload):
    """The setting a record hands out is one of its table, with the time given."""
    with open(os.path.join(tune.TUNED_DIR, f"{workload}.json")) as f:
        d = json.load(f)
    for rec in d["by_precision"].values():
        times = [t["ms"] for t in rec["table"]
                 if {k: v for k, v in t.items() if k != "ms"} == rec["best"]]
        assert rec["best_ms"] in times
