"""The line that bench.py prints on stdout: every key that describes the headline, the other configurations in short, and short enough to
survive where only the last few thousand characters of the output are kept."""
import json

import bench

KEYS = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config", "timing", "roofline")


def test_the_line_is_short_and_complete():
    layer = {"workload": "28672->8192 INT4 r=128 M=256", "mode": "m" * 190, "us_median": 152.778, "us_min": 152.552, "us_mean": 152.706, "bound": "mfma",
             "branch_overhead_pct": 10.83}
    layer_set = {"workload": "Llama2-7B-shaped decode layer set, 7 linears per step, INT3, rank 64, M=16", "us_per_step_median": 53.76, "branch_overhead_pct": 11.2}
    record = {k: "x" * 300 for k in KEYS}
    record.update({k: "y" * 1000 for k in bench.DETAILS}, configs=[layer] * 27 + [layer_set] * 4)
    text = json.dumps(bench.headline(record))
    line = json.loads(text)
    assert all(line[k] == record[k] for k in KEYS)
    assert line["configs"][0] == ["28672->8192 INT4 r=128 M=256", 152.778, 10.83] and line["configs"][-1][1] == 53.76 and len(line["configs"]) == 31
    assert len(text) < 8000
