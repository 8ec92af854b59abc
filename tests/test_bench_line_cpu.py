"""The benchmark's printed line: every figure of its contract, and short."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

CONTRACT = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
            "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline")


def test_the_line_is_short_and_whole():
    import bench
    with open(os.path.join(ROOT, "profiles", "bench_hbm_scale.json")) as f:
        record = json.loads(f.read())
    line = bench.headline(record)
    assert all(line[k] == record[k] for k in CONTRACT if k != "cpu_baseline")
    assert line["cpu_baseline"]["value"] == record["cpu_baseline"]["value"]
    assert set(line) == set(record)  # a headline of every section
    assert len(json.dumps(line)) < 6000


def test_sections_left_out_are_left_out():
    import bench
    assert bench.headline({"metric": "m", "value": 1.0}) == {"metric": "m", "value": 1.0}
