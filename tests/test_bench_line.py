"""The line that bench.py prints, made from the whole record of a run: short enough to be kept, with the fields that are read from it."""
import json
import os

import bench


def test_the_printed_line_is_short_and_whole():
    record = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "bench_record.json")))
    line = bench.brief(record)
    assert len(json.dumps(line)) <= bench.LINE_CHARS
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data",
              "config", "pct_of_hbm_peak", "roofline", "roofline_prefill", "prefill", "fusion", "kv_append", "cpu_baseline", "quantize"):
        assert line[k] == record[k], k
    assert set(line["configs"]) == set(record["configs"]) and all(line["configs"].values())
    assert line["configs"]["cfg5_dense14b"]["group_64"]["prefill_M2048"]["frac"] == record["configs"]["cfg5_dense14b"]["group_64"]["prefill_M2048"]["layer"]["frac"]
    assert line["small_batch_us"]["M=16"]["qkv"] == record["small_batch"]["per_M"]["M=16"]["qkv"]["us"]


def test_sections_that_did_not_run_are_left_out():
    record = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "bench_record.json")))
    least = {k: record[k] for k in ("metric", "value", "unit", "config", "roofline", "quantize")}
    least["configs"] = {"cfg2_chatglm2_decode": {"workload": "w", "roofline": record["roofline"]}}
    assert set(bench.brief(least)) == set(least)
