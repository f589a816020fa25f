"""The benchmark's result line: the fields it promises, short enough to be
recorded whole however many sections a run measured."""
from __future__ import annotations

import json

import bench

FIELDS = {"metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
          "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"}


def test_result_line_holds_the_headline_and_stays_short():
    lat = {"p50_us": 3.3612345, "mean_us": 3.4, "p99_us": 3.6, "span_p50_us": 2.1, "stamp_free_mean_us": 3.2}
    many = {f"case_{i}": {"p50_us": 1.0 + i, "p99_us": 2.0 + i, "grid": 224, "threads": 512} for i in range(400)}
    result = {"headline": {**lat, "exchange_probe": lat, "formats": many}, "floor": {"floor": lat, "composed_p50_us": 2.1},
              "bw": {bench.BW_ALGO: {"gbps": 6500.0, "grid": 1000, "threads": 128, "kernel_us": 315.0,
                                     "algorithmic_bytes": 2e9}, **many},
              "copy": {"streaming_probe": {"copy": {"gbps": 6000.0}}}, "c3": {"auto": {"p50_us": 9.4, "frac_of_bound": 0.3,
              "bound_us": 3.8}, "auto_sentinel_allowed": {"p50_us": 9.4, "frac_of_bound": 0.3}, **many},
              "c5": many, "rooted": many, "scratch": many, "cpu": {"value": 80.0, "unit": "us", "cores": 1}}
    text = json.dumps(bench.result_line(result, 20, 5))
    assert len(json.dumps(result)) > 100_000 and len(text) < 6000
    line = json.loads(text)
    assert FIELDS <= set(line)
    assert (line["value"], line["steps"], line["warmup"], line["n_gpus"]) == (3.361, 20, 5, 1)
    assert line["roofline"]["latency"]["p50_us"] == 3.361
