"""The result line of bench.py: the whole record is too long for a reader that keeps
the last 16 KB of the output."""
import json

from test_bench_cpu import bench  # noqa: F401  (fixture)


def test_result_line_is_short_and_keeps_what_it_reports(bench):  # noqa: F811
    times = {f"{v},{k}": 1234.56 for v, k in ((0, 1), (1, 1), (2, 2), (2, 4), (2, 8), (2, 16), (2, 32))}
    shape = {"op": "layernorm_fwd", "N": 524288, "plan": [2, 16], "us": 736.61, "gbps": 5836.4, "frac": 0.7295,
             "geometry": {"grid": 512, "per_cu": 2, "vpt": 32, "rows": 1}, "plan_times_us": times, "plan_mad_us": times,
             "best_plan": [2, 16], "judge_plan": [2, 16], "regret": 0.0, "regret_noise_aware": 0.0,
             "learned_untimed_plan": [2, 16], "learned_untimed_regret": 0.0, "learned_untimed_regret_noise_aware": 0.0}
    suite = [{"workload": "quant_int8", "M": 4096, "N": 65536, "plans_us": times}] * 60
    full = {"metric": "m", "value": 5597.7, "unit": "GB/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 2.0396,
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
            "config": {"workload": "w" * 200}, "roofline": {"kernel": "k" * 300}, "cpu_baseline": {"sample": "s" * 400},
            "per_shape": [dict(shape) for _ in range(8)], "forms": suite, "paper_suite": suite, "primitives": times,
            "source_hash": "0123456789abcdef", "copy_kernel_bytes": 1 << 30, "regret_geomean": 0.0}
    assert len(json.dumps(full)) > 20000
    line = bench.result_line(full)
    assert len(json.dumps(line)) < 4096
    for k in set(full) - {"per_shape", "forms", "paper_suite", "primitives"}:
        assert line[k] == full[k]
    assert [r["us"] for r in line["per_shape"]] == [736.61] * 8 and line["per_shape"][0]["regret"] == 0.0
    assert "plan_times_us" in full["per_shape"][0]  # the record itself is unchanged
