"""The benchmark's result line: one line of strict JSON of a few KB."""
import json

import bench


def strict(text):
    def refuse(name):
        raise ValueError(name)
    return json.loads(text, parse_constant=refuse)


def test_line_is_short_and_strict():
    run = {"policy": "joint", "p95": float("nan"), "trace": [{"k": i, "sample": 0.1} for i in range(2000)]}
    out = {"metric": "m", "value": 1.5, "unit": "tok/s", "n_gpus": 1, "corun": {"decode_ms": float("inf"), "steps": 0},
           "budgets": {"64": {"ms": 1.0}}, "policy_model": [0.5] * 1000,
           "serving_loop": {"runs": [run] * 18, "mean_over_seeds": [{"policy": "joint", "p95": 2.0}]}, "dit_corun": None}
    line, details = bench.result_line(out)
    assert "\n" not in line and len(line) < 8000
    got = strict(line)
    assert got["value"] == 1.5 and got["corun"] == {"decode_ms": None, "steps": 0} and got["dit_corun"] is None
    assert got["serving_loop"] == {"mean_over_seeds": [{"policy": "joint", "p95": 2.0}]} and "policy_model" not in got
    assert len(strict(details)["serving_loop"]["runs"]) == 18
