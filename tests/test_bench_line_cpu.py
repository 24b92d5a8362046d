"""The line that bench.py prints."""
import importlib.util
import json
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_printed_line_is_short_and_complete():
    """Readers keep the last 8000 bytes of the output: tables by kernel and by layer stay out of the line."""
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    third = 1000.0 / 3
    row = {"ms_per_step": third, "launches": 10, "tflops": third, "note": "x" * 40}
    out = {k: third for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better",
                              "scaling", "vs_baseline", "dtype", "data", "config")}
    out.update({"kernels": {f"igemm_dgrad_ws_{i}": row for i in range(60)},
                "hbm_bound_layers_hot_cold": [{p: row for p in ("fwd", "dgrad", "wgrad")} for _ in range(20)],
                "roofline": {"kernel": "k", "frac": third, "next_kernels": [row] * 20},
                "res3_res4_3x3_isolated": {"pct_peak_all": third, "distinct_layers": [row] * 30},
                "second_workload": {"ms": third, "groups": {str(i): row for i in range(30)}},
                "per_config": [{"config": i, "workload": "w" * 400, "tflops": third, "oracle_sample": "s" * 400} for i in range(4)],
                "fused_epilogue": None})
    line = json.dumps(bench.printed(out))
    assert len(line) < 1500 and json.loads(line)["ms_per_step"] == 333.33
    assert json.loads(line)["roofline"] == {"kernel": "k", "frac": 333.33} and len(json.loads(line)["per_config"]) == 4
    assert "next_kernels" in out["roofline"] and "kernels" in out       # the report keeps them
