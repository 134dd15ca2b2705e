"""The benchmark's printed line keeps the contract's fields whole and stays short, whatever the whole
record holds."""
import json

import bench

CONTRACT = {"metric": "m" * 80, "value": 28.6e6, "unit": "knot-evals/s", "n_gpus": 1, "steps": 20,
            "warmup": 5, "ms_per_step": 0.00447, "higher_is_better": True, "scaling": "weak",
            "vs_baseline": None, "dtype": "f32", "data": "synthetic",
            "config": {"workload": "w" * 90, "robot": "chain7", "knots": 128, "lanes_per_knot": 16}}


def full_record():
    times = {"us_per_step": 123.456, "kernel_avg_us": 123.456}
    rate = {"p50_us": 123.456, "p99_us": 1234.567, "p50_split_us": {"kernel": 1.0},
            "per_model": {k: {"requests": 1} for k in "abc"}}
    modes = ("two_calls", "batch_call", "graph", "one_launch", "persistent", "per_robot",
             "graph_one_launch", "graph_persistent", "tuned")
    return {**CONTRACT, "roofline": {f"field_{k}": 123.456789 for k in range(16)},
            "plain": {"value": 1.0e6, "unit": "knot-evals/s", "ms_per_step": 0.02, "note": "n" * 100},
            "fused_vs_plain": 5.4, "builds": {f"grid_fdgrad_{k}_halves": times for k in range(6)},
            "tuned": {str(1 << k): 4 for k in range(8)},
            "io_inclusive": {"wall_ms_per_call": 0.02, "pageable": {"wall_ms_per_call": 0.03},
                             "mapped": {k: {"wall_ms_per_call": 0.02} for k in ("copy_kernel", "direct")}},
            "io_sweep": {str(k): "x" * 1000 for k in range(10)},
            "sweep": {str(1 << k): {"ms_per_step": 0.0131, "note": "x" * 100} for k in range(10, 17)},
            "mixed": {"workload": "w" * 100,
                      **{p: {m: times for m in modes} for p in ("64+37", "256+181", "1024+613")}},
            "autograd": {k: 123.456789 for k in ("a", "b", "c", "d")},
            "served": {"workload": "w" * 100, "tuned_builds": {"chain7": {"16": "k" * 20}},
                       **{m: {**{str(r): rate for r in (5000, 10000, 20000, 40000)}, "launches": 7}
                          for m in ("batched", "batched_in_place", "batched_copy_engines",
                                    "per_request_plain")}},
            "cpu_baseline": {"value": 1.2e6, "unit": "knot-evals/s", "cores": 16, "kind": "oracle",
                             "sample": "s" * 200, "sweep": {str(k): "x" * 200 for k in range(20)}}}


def test_line_is_short_and_holds_the_contract():
    record = full_record()
    line = bench.headline(record)
    assert all(line[k] == v for k, v in CONTRACT.items())
    assert line["roofline"] == record["roofline"]
    assert line["served_us"]["batched_in_place"]["20000"] == [123.5, 1234.6]
    assert line["mixed_us"]["256+181"]["persistent"] == 123.456
    assert set(line["cpu_baseline"]) == {"value", "unit", "cores", "kind", "sample"}
    text = json.dumps(line)
    assert len(text) < 6000 and "\n" not in text


def test_line_of_a_short_run():
    assert bench.headline(dict(CONTRACT)) == CONTRACT
