"""The line that bench.py prints, made from the whole record of a run: short enough to be kept, with the fields that are read from it."""
import json
import os
import re

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


def test_kernel_summaries_name_every_matmul_kernel():
    csrc = os.path.join(os.path.dirname(bench.__file__), "paper_2403_20041_amd", "csrc")
    names = set()
    for f in os.listdir(csrc):
        if f.endswith(".hip"):
            names |= set(re.findall(r"\b((?:gemv|gemm|splitk)\w*_kernel)\(", open(os.path.join(csrc, f)).read()))
    assert len(names) >= 7
    for n in names:
        assert re.search(bench.OUR_KERNELS, n), n
        mangled = "_ZN4e0m412_GLOBAL__N_1%d%sILi3ELi2EEEvPKDF16_" % (len(n), n)
        assert bench._short_kernel_name(mangled).startswith(n + "<3"), n
